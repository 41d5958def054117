"""Tridiagonalisation and divide and conquer (orders up to 1280): edges of its tiers (leaves of 16, one CU's panels at 256
and 768 columns, vectors per workgroup at 320 and 640), spectra that deflate or cluster, and what must come out exactly.

Bounds as in test_gpu_eigen.py (a backward stable fp32 method: a small multiple of 6e-8 ||M|| on the eigenvalues, on
||M Q - Q D|| / ||M||_F, and an orthogonality defect of a few hundred roundings at most)."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import paper_2206_15143_amd as kf

pytestmark = pytest.mark.gpu


def _eigen(mats):
    """One layer per pair of matrices."""
    n = len(mats)
    descs = [kf.LayerDesc.linear(a.shape[0], g.shape[0], False, kf.KFAC_F32) for a, g in mats]
    low = lambda m: gu.to_dev(np.where(np.tril(np.ones_like(m)) > 0, m, np.nan).astype(np.float32))  # noqa: E731
    A, G = [low(a) for a, _ in mats], [low(g) for _, g in mats]
    QA, QG = [torch.full_like(a, float("nan")) for a in A], [torch.full_like(g, float("nan")) for g in G]
    vA = [torch.full((len(a),), float("nan"), device=gu.DEV) for a in A]
    vG = [torch.full((len(g),), float("nan"), device=gu.DEV) for g in G]
    info = torch.full((2 * n,), -1, dtype=torch.int32, device=gu.DEV)
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, [1] * n, [1] * n, [1] * n))
    kf.kfac_eigen_batched(descs, A, G, QA, vA, QG, vG, info, ws)
    torch.cuda.synchronize()
    out = []
    for i in range(n):
        out.append((mats[i][0], QA[i].cpu().numpy(), vA[i].cpu().numpy()))
        out.append((mats[i][1], QG[i].cpu().numpy(), vG[i].cpu().numpy()))
    return out, info.cpu().numpy()


def _check(M, Q, v, tag):
    """Numbers below 2^-126 are rounded to multiples of q = 2^-149: n columns, each rounding n x n entries by at most q, add
    n^2 q to what the relative bounds allow."""
    n = len(M)
    Md, Qd, vd = M.astype(np.float64), Q.astype(np.float64), v.astype(np.float64)
    Md = np.tril(Md) + np.tril(Md, -1).T
    ref = np.linalg.eigvalsh(Md)
    top = max(abs(ref[0]), abs(ref[-1]), 1e-300)
    e_val = np.abs(np.sort(vd) - ref).max() / top
    e_orth = np.linalg.norm(Qd.T @ Qd - np.eye(n)) / np.sqrt(n)
    e_res = np.linalg.norm(Md @ Qd - Qd * vd) / max(np.linalg.norm(Md), 1e-300)
    print(f"{tag}: eigenvalues {e_val:.2e} orthogonality {e_orth:.2e} residual {e_res:.2e}", flush=True)
    q = n * n * 2.0 ** -149
    assert e_val <= 2e-6 + q / top, tag
    assert e_orth < 1e-4, tag
    assert e_res < 2e-5 + q / max(np.linalg.norm(Md), 1e-300), tag


def _factor(n, rows, seed, relu=True):
    x = np.random.default_rng(seed).standard_normal((rows, n))
    x = np.maximum(x, 0) if relu else x
    return (0.95 * np.eye(n) + 0.05 * x.T @ x / 3).astype(np.float32)


def _with_spectrum(lam, seed):
    n = len(lam)
    q, _ = np.linalg.qr(np.random.default_rng(seed).standard_normal((n, n)))
    m = (q * lam) @ q.T
    return ((m + m.T) / 2).astype(np.float32)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 18, 31, 32, 33, 34, 63, 65, 97, 128, 129, 255, 257, 258, 319, 321, 577, 640, 641, 768, 769, 1025, 1280])
def test_orders(n):
    (a, g), info = _eigen([(_factor(n, 3 * n, n), _factor(7 + n % 31, 50, n + 1))])
    assert list(info) == [0, 0]
    _check(*a, f"n={n}")
    _check(*g, "G")


SPECTRA = {
    "rank deficient": lambda n: _factor(n, n // 3, 5, relu=False),
    "two values": lambda n: _with_spectrum(np.r_[np.full(n // 2, 1.0), np.full(n - n // 2, 3.0)], 6),
    "graded": lambda n: _with_spectrum(np.geomspace(1e-6, 1.0, n), 7),
    "clusters": lambda n: _with_spectrum(np.repeat(np.arange(1.0, 9.0), (n + 7) // 8)[:n] + 1e-6 * np.arange(n), 8),
    "indefinite": lambda n: _with_spectrum(np.linspace(-1.0, 1.0, n), 9),
    "one large": lambda n: (np.eye(n) + 100.0 * np.ones((n, n))).astype(np.float32),
    "tridiagonal": lambda n: (2 * np.eye(n) + np.eye(n, k=1) + np.eye(n, k=-1)).astype(np.float32),
    "wilkinson": lambda n: (np.diag(np.abs(np.arange(n) - n // 2).astype(float)) + np.eye(n, k=1) + np.eye(n, k=-1)).astype(np.float32),
    "blocks": lambda n: np.kron(np.eye((n + 9) // 10), _factor(10, 30, 10))[:n, :n].astype(np.float32),
    "tiny": lambda n: (1e-20 * _factor(n, 2 * n, 11)).astype(np.float32),
    "huge": lambda n: (1e25 * _factor(n, 2 * n, 12)).astype(np.float32),
    "dense among diagonal": lambda n: _among_diagonal(n),
    "zero": lambda n: np.zeros((n, n), dtype=np.float32),
}


@pytest.mark.parametrize("kind", sorted(SPECTRA))
@pytest.mark.parametrize("n", [50, 145, 300, 801])
def test_spectra(kind, n):
    m = SPECTRA[kind](n)
    (a, _), info = _eigen([(m, np.eye(3, dtype=np.float32))])
    assert list(info) == [0, 0]
    _check(*a, f"{kind} n={n}")


def _among_diagonal(n):
    """Columns with nothing to reduce before and behind those with something, inside a panel of the reduction and across."""
    m = np.diag(np.linspace(1.0, 2.0, n)).astype(np.float32)
    for at, size in ((n // 5, n // 4), (n - n // 7 - 3, n // 7)):
        m[at:at + size, at:at + size] = _factor(size, 2 * size, size)
    return m


def _dead(n, at, value, count=1):
    """Rows and columns at .. at + count - 1 of a factor whose features stopped firing: every update multiplied them by the
    decay, and rounding keeps them at a few multiples of 2^-149; entries that were zero stay zero."""
    m = _factor(n, 2 * n, n + at)
    for i in range(at, at + count):
        m[i, :] = m[:, i] = value
        m[i, ::3] = m[::3, i] = 0.0
    for i in range(at, at + count):
        m[i, i] = 2 * value
    return m


SUBNORMAL = {
    "first feature dead": lambda n: _dead(n, 0, 1.3e-44),
    "first feature nearly dead": lambda n: _dead(n, 0, 1e-39),
    "middle feature dead": lambda n: _dead(n, n // 2, 1.3e-44),
    "last feature dead": lambda n: _dead(n, n - 1, 1.3e-44),
    "last third dead": lambda n: _dead(n, n - n // 3, 1.3e-44, n // 3),
    "first third dead": lambda n: _dead(n, 0, 1.3e-44, n // 3),
    "one subnormal pair": lambda n: (np.diag(np.arange(1.0, n + 1)) + 1e-40 * (np.eye(n, k=3) + np.eye(n, k=-3)) * (np.arange(n) < 4)
                                     * (np.arange(n)[:, None] < 4)).astype(np.float32),
    "all subnormal": lambda n: (1e-40 * _factor(n, 2 * n, 13)).astype(np.float32),
    "largest": lambda n: (_factor(n, 2 * n, 14) * (1e38 / np.linalg.norm(_factor(n, 2 * n, 14), 2))).astype(np.float32),
}


@pytest.mark.parametrize("kind", sorted(SUBNORMAL))
@pytest.mark.parametrize("n", [40, 145, 300, 800])
def test_ends_of_the_range(kind, n):
    """A column's reflector is scaled by the reciprocal of a norm that may lie outside the range of fp32 although the column does
    not: below 2.9e-39 the reciprocal is infinite, above 8.5e37 it has few bits left.  (With many dead features the reduction finds
    their direction in steps whose reflectors have hundreds of equal entries, and sums of equal terms round the same way each
    time: orthogonality 1.7e-5 at order 800, below n 2^-24.)"""
    m = SUBNORMAL[kind](n)
    (a, _), info = _eigen([(m, np.eye(3, dtype=np.float32))])
    assert list(info) == [0, 0]
    assert np.isfinite(a[1]).all() and np.isfinite(a[2]).all()
    _check(*a, f"{kind} n={n}")


@pytest.mark.parametrize("n", [20, 90, 577])
def test_diagonal_is_exact_and_in_place(n):
    d = np.random.default_rng(n).permutation(n).astype(np.float32) // 3
    (a, g), info = _eigen([(np.diag(d), np.eye(n, dtype=np.float32))])
    assert list(info) == [0, 0]
    assert np.array_equal(a[1], np.eye(n)) and np.array_equal(a[2], d)
    assert np.array_equal(g[1], np.eye(n)) and np.array_equal(g[2], np.ones(n))


def test_many_matrices_of_mixed_orders():
    """More than one launch's table (256), every tier at once, one matrix beyond the range of the method; the second table, the
    smallest of 279, holds nothing but leaves."""
    sizes = [(577, 64), (1300, 20), (289, 33), (145, 200)] + [(30 + 5 * (i % 40), 10 + i % 60 if i % 3 else 1 + i % 16) for i in range(136)]
    assert sorted(n for s in sizes for n in s)[23] <= 16 and len(sizes) == 140
    mats = [(_factor(a, 2 * a, i), _factor(g, 2 * g, 500 + i)) for i, (a, g) in enumerate(sizes)]
    out, info = _eigen(mats)
    assert not info.any()
    for m, q, v in out:
        _check(m, q, v, f"n={len(m)}")


def test_not_finite_input_ends():
    """No result to speak of, but every loop of the method is bounded and the others of the call are not affected."""
    bad = _factor(150, 300, 1)
    bad[40, 7] = np.nan
    inf = _factor(150, 300, 2)
    inf[3, 3] = np.inf
    good = _factor(150, 300, 3)
    out, _ = _eigen([(bad, good), (inf, good)])
    _check(*out[1], "beside NaN")
    _check(*out[3], "beside infinity")
