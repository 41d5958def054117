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
    new = _factor(c, h, w, b, bias, x, A0 + np.triu(A0.T, 1))
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
