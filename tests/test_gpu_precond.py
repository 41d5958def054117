"""The one-launch form of the two-sided product (layers with a dimension of at most 64) at the sizes where it can go wrong:
edges of the 16-wide MFMA tiles and of the 32- and 64-wide workgroup tiles, one column past them, depths below one chunk
and of many, either dimension the small one; groups of eight layers and the rest behind them; outputs in place.

Tolerance: fp32 sums of at most K terms in a few partial sums carry about sqrt(K) 2^-24 of the product of the norms
(2e-6 at K = 2049); 1e-5 leaves a factor of five."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import paper_2206_15143_amd as kf

pytestmark = pytest.mark.gpu


def _sym(d, rng):
    m = rng.standard_normal((d, d)) / np.sqrt(d)
    return (m + m.T + np.diag(rng.random(d) + 0.5)).astype(np.float32)


def _layers(shapes, seed):
    rng = np.random.default_rng(seed)
    out = []
    for dA, dG in shapes:
        A, G, W = _sym(dA, rng), _sym(dG, rng), rng.standard_normal((dG, dA)).astype(np.float32)
        out.append((A, G, W, G.astype(np.float64) @ W.astype(np.float64) @ A.astype(np.float64)))
    return out


def _desc(dA, dG):
    return kf.LayerDesc.linear(dA - 1, dG, True, kf.KFAC_F32) if dA > 1 else kf.LayerDesc.linear(1, dG, False, kf.KFAC_F32)


def _run(shapes, layers, in_place=False):
    descs = [_desc(*s) for s in shapes]
    A, G, W = ([gu.to_dev(l[k]) for l in layers] for k in range(3))
    out = W if in_place else [torch.full(l[2].shape, float("nan"), device=gu.DEV) for l in layers]
    n = len(shapes)
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, [1] * n, [1] * n, [1] * n))
    kf.kfac_precondition_batched(descs, A, G, W, out, ws)
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


SHAPES = [(1, 1), (16, 16), (17, 15), (32, 33), (33, 32), (64, 64), (65, 64), (64, 65), (66, 17), (129, 48), (31, 193),
          (577, 64), (64, 577), (300, 1), (2049, 10), (10, 1000), (67, 62)]


@pytest.mark.parametrize("shape", SHAPES)
def test_one_layer(shape):
    layers = _layers([shape], 11)
    got = _run([shape], layers)[0]
    err = gu.rel_fro(got, layers[0][3])
    print(shape, f"{err:.2e}")
    assert err < 1e-5


@pytest.mark.parametrize("reps", [1, 4])
def test_many_layers_and_in_place(reps):
    """17 reps layers (two groups of eight and a rest; from 256 tiles on the 64-wide tiles), two wide ones among them."""
    shapes = (SHAPES + [(200, 130), (577, 64), (577, 64), (300, 64)]) * reps + [(577, 64)] * (30 * (reps - 1))
    layers = _layers(shapes, 12)
    a = _run(shapes, layers)
    b = _run(shapes, layers, in_place=True)
    for s, l, x, y in zip(shapes, layers, a, b):
        assert gu.rel_fro(x, l[3]) < 1e-5, s
        assert gu.rel_fro(y, l[3]) < 1e-5, s


def test_infinite_column_stays_in_its_columns():
    """An infinite entry of A_inv (an inverse that failed) reaches the columns it belongs to and no others."""
    shape = (129, 40)
    A, G, W, _ = _layers([shape], 13)[0]
    A = A.copy()
    A[5, 70] = np.inf
    got = _run([shape], [(A, G, W, None)])[0]
    keep = [c for c in range(129) if c != 70]
    ref = (G.astype(np.float64) @ W.astype(np.float64) @ A.astype(np.float64)[:, keep])
    assert not np.isfinite(got[:, 70]).any()
    assert gu.rel_fro(got[:, keep], ref) < 1e-5


def _eigen_layers(shapes, seed):
    rng = np.random.default_rng(seed)
    out = []
    for dA, dG in shapes:
        QA, QG = (np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32) for d in (dA, dG))
        vA, vG = ((rng.random(d) + 0.5).astype(np.float32) for d in (dA, dG))
        W = rng.standard_normal((dG, dA)).astype(np.float32)
        a, g = QA.astype(np.float64), QG.astype(np.float64)
        out.append((QA, vA, QG, vG, W, g @ ((g.T @ W @ a) / (np.outer(vG, vA).astype(np.float64) + 0.1)) @ a.T))
    return out


@pytest.mark.parametrize("turn", [0, 1, 2, 3])
def test_eigen_form_with_outputs_over_gradients(turn):
    """Wide and narrow layers in one call, every output in the gradient buffer of the layer `turn` places on (0: its own): all
    gradients are read before an output is stored."""
    shapes = [(200, 130), (520, 50), (130, 200), (50, 520)]
    layers = _eigen_layers(shapes, 21)
    n = len(shapes)
    QA, vA, QG, vG, W = ([gu.to_dev(l[k]) for l in layers] for k in range(5))
    out = [W[(i + turn) % n].view(shapes[i][1], shapes[i][0]) for i in range(n)]
    descs = [_desc(*s) for s in shapes]
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, [1] * n, [1] * n, [1] * n))
    kf.kfac_precondition_eigen_batched(descs, QA, vA, QG, vG, 0.1, W, out, ws)
    torch.cuda.synchronize()
    for s, l, o in zip(shapes, layers, out):
        assert gu.rel_fro(o.cpu().numpy(), l[5]) < 1e-5, s


def test_outputs_over_inverses_of_g():
    """G_inv of a layer may be reused for another layer's output: two products read all of them before an output is stored, and
    so must a call of more layers than one launch of the fused form holds (128)."""
    n, d = 160, 64
    rng = np.random.default_rng(31)
    A, G = [_sym(d, rng) for _ in range(n)], [_sym(d, rng) for _ in range(n)]
    W = [rng.standard_normal((d, d)).astype(np.float32) for _ in range(n)]
    dev = [[gu.to_dev(x) for x in xs] for xs in (A, G, W)]
    out = [dev[1][128 + i] if i < 32 else torch.full((d, d), float("nan"), device=gu.DEV) for i in range(n)]
    descs = [_desc(d, d)] * n
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, [1] * n, [1] * n, [1] * n))
    kf.kfac_precondition_batched(descs, *dev, out, ws)
    torch.cuda.synchronize()
    for i in range(n):
        ref = G[i].astype(np.float64) @ W[i].astype(np.float64) @ A[i].astype(np.float64)
        assert gu.rel_fro(out[i].cpu().numpy(), ref) < 1e-5, i


def test_eigen_form_of_many_layers():
    """More transposes than one launch's table holds (256) and more narrow layers (128), wide ones among them."""
    shapes = [SHAPES[i % len(SHAPES)] if i % 17 else (70 + i, 90) for i in range(150)]
    shapes = [s if max(s) < 1000 else (100, 30) for s in shapes]
    layers = _eigen_layers(shapes, 22)
    n = len(shapes)
    QA, vA, QG, vG, W = ([gu.to_dev(l[k]) for l in layers] for k in range(5))
    out = [torch.full_like(w, float("nan")) for w in W]
    descs = [_desc(*s) for s in shapes]
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, [1] * n, [1] * n, [1] * n))
    kf.kfac_precondition_eigen_batched(descs, QA, vA, QG, vG, 0.1, W, out, ws)
    torch.cuda.synchronize()
    for s, l, o in zip(shapes, layers, out):
        assert gu.rel_fro(o.cpu().numpy(), l[5]) < 1e-5, s
