"""Factors of wide 3x3 convolutions from autocorrelations of a padded copy: channel counts that fill no tile and no block of
64, maps from 7 x 7 up that are odd, flat or tall, one image and many, K slices with remainders, with and without bias.

Against float64, and against the route over the patch matrix: the sums run over the same products (12.5 of 40.5 C^2 of
them per position), so the error is that of fp32 sums of K terms on either, below 1e-5 for the sizes here, and the new route's
must not exceed 1.5 times the other's (plus 1e-7: both round the factor's entries)."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import paper_2206_15143_amd as kf

pytestmark = pytest.mark.gpu

CASES = [  # channels, h, w, batch, bias, relu
    (20, 28, 28, 3, 1, True), (24, 9, 33, 2, 0, False), (28, 32, 32, 1, 1, True), (64, 56, 56, 2, 1, True), (64, 65, 70, 1, 1, True), (68, 7, 7, 3, 0, True), (96, 9, 7, 3, 1, False),
    (100, 6, 9, 2, 1, True), (128, 4, 40, 2, 1, True), (128, 14, 14, 8, 1, True), (128, 28, 28, 4, 0, True),
    (132, 30, 4, 2, 1, False), (256, 7, 7, 8, 1, True), (512, 8, 8, 2, 1, True),
]


def _factor(c, h, w, b, bias, x, A0):
    d = kf.LayerDesc.conv2d(c, 4, 3, 1, 1, bool(bias), kf.KFAC_F32)
    n = 9 * c + bias
    A = gu.to_dev(A0)
    G = torch.zeros(4, 4, device=gu.DEV)
    g = torch.zeros(b, 4, h, w, device=gu.DEV)
    ws = gu.workspace(kf.kfac_workspace_bytes(d, b, h, w))
    kf.kfac_update_factors(d, gu.to_dev(x), g, b, h, w, 1.0 / b, 1.0, 0.9, A, G, ws)
    torch.cuda.synchronize()
    assert A.shape == (n, n)
    return A.cpu().numpy()


@pytest.mark.parametrize("case", CASES)
def test_wide_conv_factor(case):
    c, h, w, b, bias, relu = case
    rng = np.random.default_rng(c + h + w)
    x = rng.standard_normal((b, c, h, w)).astype(np.float32)
    x = np.maximum(x, 0) if relu else x
    n = 9 * c + bias
    A0 = np.tril(rng.standard_normal((n, n))).astype(np.float32)
    cols = torch.nn.functional.unfold(torch.from_numpy(x).double(), 3, padding=1)     # [b, 9 c, h w]
    p = cols.permute(0, 2, 1).reshape(-1, 9 * c)
    if bias:
        p = torch.cat([p, torch.ones(len(p), 1, dtype=torch.float64)], 1)
    low = A0.astype(np.float64)
    ref = 0.9 * (low + np.tril(low, -1).T) + 0.1 / b * (p.T @ p).numpy()
    kf.kfac_tune("corrw_min_gain", 0)                     # most of these layers are too small to take the route by themselves
    try:
        new = _factor(c, h, w, b, bias, x, A0 + np.triu(A0.T, 1))
    finally:
        kf.kfac_tune("corrw_min_gain", 42)
    kf.kfac_tune("use_corr3", 0)
    try:
        old = _factor(c, h, w, b, bias, x, A0 + np.triu(A0.T, 1))
    finally:
        kf.kfac_tune("use_corr3", 1)
    e_new, e_old = gu.rel_fro(new, ref), gu.rel_fro(old, ref)
    print(case, f"autocorrelations {e_new:.2e}, patch matrix {e_old:.2e}")
    assert e_new < 1e-5
    assert e_new < 1.5 * e_old + 1e-7
    assert np.array_equal(new, new.T)


def _routes(layers):
    """The kernels that one call over layers (channels, map, batch) launches for their factors."""
    descs = [kf.LayerDesc.conv2d(c, 4, 3, 1, 1, True, kf.KFAC_F32) for c, _, _ in layers]
    b, h = [l[2] for l in layers], [l[1] for l in layers]
    x = [torch.ones(n, c, s, s, device=gu.DEV) for c, s, n in layers]
    g = [torch.zeros(n, 4, s, s, device=gu.DEV) for _, s, n in layers]
    A = [torch.zeros(9 * c + 1, 9 * c + 1, device=gu.DEV) for c, _, _ in layers]
    G = [torch.zeros(4, 4, device=gu.DEV) for _ in layers]
    ws = gu.workspace(kf.kfac_workspace_bytes_batched(descs, b, h, h))
    one = [1.0] * len(layers)
    kf.kfac_timing_enable(True)
    try:
        kf.kfac_update_factors_batched(descs, x, g, b, h, h, one, one, 0.0, A, G, ws)
        launches = kf.kfac_timing_collect()
    finally:
        kf.kfac_timing_enable(False)
    for a, (c, s, n) in zip(A, layers):                   # all ones: the corner of the bias counts the positions, tap (1, 1) too
        assert float(a[-1, -1]) == n * s * s and float(a[4, 4]) == n * s * s
    names = {"im2col": "patches", "syrk_conv3": "fused", "syrk_split": "copies"}     # (no factor here is split otherwise)
    return {names[k] for k, v in launches.items() if k in names and v[1]}


@pytest.mark.parametrize("layers, routes", [
    ([(36, 14, 8)], {"patches"}), ([(36, 28, 128)], {"copies"}),      # a layer by itself: by its work
    ([(36, 14, 8)] * 3, {"patches"}), ([(36, 28, 8)] * 12, {"copies"}),    # layers of a call together
    ([(20, 28, 32)], {"patches"}), ([(20, 50, 128)] * 2, {"copies"}),       # the alternative that costs least,
    ([(96, 28, 8)], {"copies"}), ([(96, 8, 1)], {"patches"}),      # those that take as long as the launches
    ([(48, 28, 8)], {"copies"}), ([(48, 8, 2)], {"fused"}),
    ([(36, 14, 8), (96, 28, 8)], {"copies"}),                      # a layer that takes the route anyway brings its launches,
    ([(48, 8, 2), (36, 14, 8), (96, 28, 8)], {"copies", "fused"}),        # but nothing to one without gain
    ([(64, 8, 8), (36, 14, 8)], {"patches"}),                      # nor one that has a kernel of its own (64 channels)
])
def test_small_calls_keep_the_other_routes(layers, routes):
    """The route costs four dependent launches: a call too small to earn them keeps the patch matrix or the fused kernel."""
    assert _routes(layers) == routes


def test_workspace_of_a_network_serves_its_layers():
    layers = [(128, 14, 8)] * 12 + [(40, 28, 16)] * 3
    descs = [kf.LayerDesc.conv2d(c, 4, 3, 1, 1, True, kf.KFAC_F32) for c, _, _ in layers]
    whole = kf.kfac_workspace_bytes_batched(descs, [l[2] for l in layers], [l[1] for l in layers], [l[1] for l in layers])
    for d, (_, s, n) in zip(descs, layers):
        assert kf.kfac_workspace_bytes(d, n, s, s) <= whole


@pytest.mark.parametrize("c, h, b", [(16, 16, 4), (64, 8, 4), (24, 15, 4), (96, 14, 4), (128, 9, 8)])
def test_border_much_larger_than_the_inside(c, h, b):
    """Entries of taps that never see a border row or column are the sum over the whole map less the border's, so they carry its
    rounding: a few 2^-24 of the geometric mean of the two channels' centre-tap entries, which hold every position (Cauchy-
    Schwarz), whatever the entry itself amounts to.  Norm-wise nothing is lost.  (A direct sum has that bound entry by entry
    only with the taps' own entries.)"""
    rng = np.random.default_rng(c + h)
    x = np.maximum(rng.standard_normal((b, c, h, h)), 0).astype(np.float32)
    for edge in (np.s_[:, :, 0], np.s_[:, :, -1], np.s_[:, :, :, 0], np.s_[:, :, :, -1]):
        x[edge] *= 1000.0
    cols = torch.nn.functional.unfold(torch.from_numpy(x).double(), 3, padding=1).permute(0, 2, 1).reshape(-1, 9 * c)
    p = torch.cat([cols, torch.ones(len(cols), 1, dtype=torch.float64)], 1)
    ref = 0.1 / b * (p.T @ p).numpy()
    kf.kfac_tune("corrw_min_gain", 0)
    try:
        got = _factor(c, h, h, b, 1, x, np.zeros_like(ref, dtype=np.float32))
    finally:
        kf.kfac_tune("corrw_min_gain", 42)
    centre = np.sqrt(np.append(np.repeat(np.diag(ref)[4:9 * c:9], 9), ref[-1, -1]))
    err = np.abs(got - ref) / np.outer(centre, centre)
    print(c, h, f"norm-wise {gu.rel_fro(got, ref):.2e}, of the centre taps {err.max():.2e}")
    assert gu.rel_fro(got, ref) < 1e-6
    assert err.max() < 16 * 2.0 ** -24
