"""The split-fp16 product kernel on its own, against float64: edges of its 256 x 128 tiles and 16-row stages, lower
triangle updates with an untouched band, operands whose columns differ wildly in size, columns that start with zeros
(the scale of the first stage does not hold and the tile is computed again), and operands whose large values only meet
tiny ones (the tile goes to the fp32 MFMA).

Bound per element: the cut into pieces leaves 2^-21 |a||b| per product, and a sum of K products that is accumulated in
fp32 loses at most K 2^-24 of sum |a||b|.
"""
import numpy as np
import pytest
import torch

import paper_2206_15143_amd as kf

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def operands(M, N, K, kind, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    A = torch.randn(K, (M + 3) // 4 * 4, generator=g, device=DEV)
    B = torch.randn(K, (N + 3) // 4 * 4, generator=g, device=DEV)
    if kind == "columns":
        A *= torch.exp(8 * torch.randn(1, A.shape[1], generator=g, device=DEV))
        B *= torch.exp(8 * torch.randn(1, B.shape[1], generator=g, device=DEV))
    elif kind == "zeros_first":
        A[:K // 3] = 0
        A[:, ::5] *= 1e-3
        B[:K // 4, : N // 2] = 0
    elif kind == "opposite":
        r = torch.linspace(-12, 12, K, device=DEV)[:, None]
        A *= torch.exp(r)
        B *= torch.exp(-r)
    elif kind == "relu":
        A.relu_()
        B.relu_()
    elif kind == "diagonal":
        n = min(K, M)
        A *= 1e-3
        A[torch.arange(n), torch.arange(n)] = 30.0
    return A, B


@pytest.mark.parametrize("M,N,K,mode,p0,p1,kind", [
    (1024, 512, 1024, 0, 0, 0, "normal"),
    (1025, 1153, 1041, 0, 0, 0, "normal"),          # one row, one column, one k past the edges
    (1023, 640, 1039, 0, 0, 0, "relu"),
    (1000, 520, 1100, 0, 0, 0, "columns"),
    (768, 512, 1030, 0, 0, 0, "zeros_first"),
    (768, 640, 1025, 0, 0, 0, "opposite"),
    (1300, 1300, 1300, 0, 0, 0, "diagonal"),
    (1025, 1025, 256, 2, 256, 512, "normal"),
    (1281, 1281, 1, 2, 1280, 1281, "normal"),
    (2305, 2305, 250, 2, 0, 512, "columns"),
    (769, 769, 256, 2, 768, 769, "opposite"),
    (128, 1090, 128, 0, 0, 0, "normal"),            # the smallest stores: rows, depth, share of the tiles filled
    (1100, 129, 129, 0, 0, 0, "columns"),
    (257, 513, 135, 0, 0, 0, "zeros_first"),
    (511, 321, 200, 0, 0, 0, "opposite"),
    (1090, 127, 128, 0, 0, 0, "relu"),              # ... and just outside: the other kernels
    (640, 512, 127, 0, 0, 0, "normal"),
])
def test_split_product(M, N, K, mode, p0, p1, kind):
    A, B = operands(M, N, K, kind, 11)
    C = torch.full((M, N), 3.0, device=DEV)
    kf.kfac_profile_gemm(A, B, C, M, N, K, A.shape[1], B.shape[1], N, mode, p0, p1)
    torch.cuda.synchronize()
    a, b = A[:, :M].double().cpu().numpy(), B[:, :N].double().cpu().numpy()
    got = C.double().cpu().numpy()
    ref, mag = a.T @ b, np.abs(a).T @ np.abs(b)
    if mode == 2:
        live = np.tril(np.ones((M, N), dtype=bool))
        live[p0:p1] = False
        live[:, p0:p1] = False
        assert np.all(got[~live] == 3.0)
        ref, mag = np.where(live, 3.0 - ref, 3.0), np.where(live, mag + 3.0, 3.0)
    bound = (2.0 ** -21 + (K + 2) * 2.0 ** -24) * mag
    worst = np.max(np.abs(got - ref) / bound)
    assert worst <= 1.0, f"error {worst:.3f} of the bound"


@pytest.mark.parametrize("d_in,d_out", [(1023, 400), (1024, 300), (2300, 200), (5000, 130)])
def test_k_slices_of_one_layer(d_in, d_out):
    """A call of one layer: its deep products are cut into slices of 40 stages and more, up to eight of them.  The same
    bound as above, twice: the first product's error passes through the second."""
    d = kf.LayerDesc.linear(d_in, d_out, True, kf.KFAC_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    n = d_in + 1
    A, G, W = (torch.randn(*s, generator=g, device=DEV) for s in ((n, n), (d_out, d_out), (d_out, n)))
    A, G = (A + A.T) / 2, (G + G.T) / 2
    work = torch.empty(kf.kfac_workspace_bytes(d, 8, 1, 1), dtype=torch.uint8, device=DEV)
    out = torch.empty(d_out, n, device=DEV)
    kf.kfac_precondition(d, A, G, W, out, work)
    torch.cuda.synchronize()
    a, b, w = A.double().cpu(), G.double().cpu(), W.double().cpu()
    mag = b.abs() @ w.abs() @ a.abs()
    bound = (2.0 ** -20 + (n + d_out + 4) * 2.0 ** -24) * mag
    worst = ((out.double().cpu() - b @ w @ a).abs() / bound).max().item()
    assert worst <= 1.0, f"error {worst:.3f} of the bound"
