"""Factors of 3x3 convolutions of 16, 32 and 64 channels: strips that do not divide the map, rows that end inside an octet of
pixels, k-steps with octets past the strip, one part and many (from 32 on the sums are shared by 16 threads), and inputs that
leave the range of the split arithmetic.

Against float64, and against the direct kernel, which sums the same products in fp32: the error is that of fp32 sums, below 1e-5
for the sizes here, and must not exceed 1.5 times the direct kernel's (plus 1e-7: both round the factor's entries)."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import paper_2206_15143_amd as kf

pytestmark = pytest.mark.gpu

CASES = [  # channels, h, w, batch, relu
    (16, 12, 8, 1, True), (16, 14, 24, 3, False), (16, 36, 20, 2, True), (16, 31, 64, 1, True), (16, 32, 32, 40, True),
    (32, 9, 12, 1, False), (32, 11, 28, 2, True), (32, 17, 60, 2, True), (32, 16, 16, 33, False),
    (64, 9, 8, 1, True), (64, 9, 36, 2, True), (64, 56, 56, 1, True), (64, 8, 8, 34, False), (64, 5, 64, 2, True),
]


def _factor(c, x):
    b, _, h, w = x.shape
    d = kf.LayerDesc.conv2d(c, 4, 3, 1, 1, True, kf.KFAC_F32)
    A = torch.zeros(9 * c + 1, 9 * c + 1, device=gu.DEV)
    G = torch.zeros(4, 4, device=gu.DEV)
    ws = gu.workspace(kf.kfac_workspace_bytes(d, b, h, w))
    kf.kfac_update_factors(d, gu.to_dev(x), torch.zeros(b, 4, h, w, device=gu.DEV), b, h, w, 1.0 / b, 1.0, 0.0, A, G, ws)
    torch.cuda.synchronize()
    return A.cpu().numpy()


def _patches(x):
    b, c, h, w = x.shape
    cols = torch.nn.functional.unfold(torch.from_numpy(x).double(), 3, padding=1).permute(0, 2, 1).reshape(-1, 9 * c)
    return torch.cat([cols, torch.ones(len(cols), 1, dtype=torch.float64)], 1)


@pytest.mark.parametrize("case", CASES)
def test_factor(case):
    c, h, w, b, relu = case
    x = np.random.default_rng(c + h + w).standard_normal((b, c, h, w)).astype(np.float32)
    x = np.maximum(x, 0) if relu else x
    p = _patches(x)
    ref = (p.T @ p).numpy() / b
    new = _factor(c, x)
    kf.kfac_tune("use_corr3", 0)
    try:
        old = _factor(c, x)
    finally:
        kf.kfac_tune("use_corr3", 1)
    e_new, e_old = gu.rel_fro(new, ref), gu.rel_fro(old, ref)
    print(case, f"autocorrelations {e_new:.2e}, direct {e_old:.2e}")
    assert e_new < 1e-5
    assert e_new < 1.5 * e_old + 1e-7
    assert np.array_equal(new, new.T)


@pytest.mark.parametrize("c", [16, 32, 64])
@pytest.mark.parametrize("value", [np.inf, np.nan, 2.0 ** 115, 2.0 ** 60])
def test_values_outside_the_split_range(c, value):
    # one pixel away from the border: the entries of its channel are what fp32 gives (infinite, NaN or large), the others
    # keep the accuracy of the ordinary path
    x = np.random.default_rng(c).standard_normal((3, c, 12, 12)).astype(np.float32)
    x[1, 5, 6, 6] = value
    p = _patches(x)
    with np.errstate(all="ignore"):
        ref = ((p.T @ p).numpy() / 3)
        ref32 = ref.astype(np.float32)
    new = _factor(c, x)
    rows = np.arange(9 * c + 1) // 9 == 5
    clean = ~rows[:, None] & ~rows[None, :]
    assert gu.rel_fro(new[clean], ref[clean]) < 1e-6
    mine = ~clean
    assert np.array_equal(np.isfinite(new[mine]), np.isfinite(ref32[mine]))
    ok = mine & np.isfinite(ref32) & (np.abs(ref32) > 0)
    if ok.any() and np.isfinite(value):
        # entries that the large value enters: relative to it, the rest of the sum is below fp32 rounding
        assert np.max(np.abs(new[ok] - ref[ok]) / np.maximum(np.abs(ref[ok]), abs(value) * 1e-3)) < 1e-5
