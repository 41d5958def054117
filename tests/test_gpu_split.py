"""The split-bf16 kernels against float64: edges of their 256 x 128 tiles and 16-row stages, lower triangle updates with
an untouched band, operands whose columns or rows differ wildly in size, large values of one operand that only meet
zeros or tiny values of the other (in all of a tile, in a few of its rows, in a quarter of its columns), the smallest
fp32 numbers, sums of the largest, infinities, NaN and values next to the largest one, and what lies between the columns of an operand and its pitch.

Bound per element: the cut into pieces leaves 2^-24 |a||b| per product, and a sum of K products that is accumulated in
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
    elif kind == "two_levels":                       # large values only meet values 1e-12 times as large
        A[K // 2:] *= 1e-12
        B[:K // 2] *= 1e-12
    elif kind == "few_columns":                      # four columns of A have their large value at a zero row of B
        A[:, 4:8] *= 1e-9
        A[0, 4:8] = 1.0
        B[0] = 0
    elif kind == "quarter":                          # one in five columns of B is tiny where A is large
        A[:K // 2] *= 1e10
        B[:K // 2, ::5] *= 1e-10
    elif kind == "features":                         # features of uneven scale: gradients ~ s, inverse ~ 1/s^2
        f = torch.exp(2 * torch.randn(K, 1, generator=g, device=DEV))
        A *= f
        B /= f
    elif kind == "one_feature":                      # one of scale 2^24, whose gradient is zero in four rows
        A[1] *= 2.0 ** 24
        B[1] *= 2.0 ** -24
        A[1, :4] = 0
    elif kind == "tiny":                             # next to the smallest fp32 numbers, down to subnormal ones
        A *= 2.0 ** -119 * torch.exp2(torch.linspace(0, -20, K, device=DEV))[:, None]
        B *= 2.0 ** 100 * torch.exp2(torch.linspace(0, 20, K, device=DEV))[:, None]
    elif kind == "tiny_rest":                        # tiny values of B beside ordinary ones that meet zeros
        A[::2] = 0
        A[1::2] *= 2.0 ** 90
        B[1::2] *= 2.0 ** -121
    elif kind == "huge":                             # sums that leave the range of the scaled accumulators
        A *= 2.0 ** 60
        B *= 2.0 ** 50
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
    (769, 769, 768, 0, 0, 0, "two_levels"),
    (1025, 513, 1040, 0, 0, 0, "two_levels"),
    (256, 769, 769, 0, 0, 0, "few_columns"),
    (1024, 512, 1024, 0, 0, 0, "quarter"),
    (256, 769, 769, 0, 0, 0, "features"),
    (512, 1025, 1025, 0, 0, 0, "features"),
    (256, 769, 769, 0, 0, 0, "one_feature"),
    (1153, 1153, 256, 2, 512, 768, "two_levels"),
    (1153, 1153, 256, 2, 512, 768, "features"),
    (512, 769, 256, 0, 0, 0, "tiny"),
    (769, 512, 1030, 0, 0, 0, "tiny_rest"),
    (1153, 1153, 256, 2, 512, 768, "tiny"),
    (257, 513, 135, 0, 0, 0, "huge"),
    (1025, 1025, 256, 2, 256, 512, "huge"),
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
    bound = (1 + K + 2) * 2.0 ** -24 * mag
    worst = np.max(np.abs(got - ref) / bound)
    assert worst <= 1.0, f"error {worst:.3f} of the bound"


@pytest.mark.parametrize("M,N,K,mode", [(257, 513, 135, 0), (1024, 512, 1024, 0), (1025, 1025, 256, 2)])
def test_infinities_nan_and_the_largest_values(M, N, K, mode):
    """What fp32 arithmetic leaves: infinities and NaN in the same places, everything else untouched by them; values that a
    rounding to 8 bits would carry to infinity keep their value."""
    A, B = operands(M, N, K, "normal", 3)
    A[5, 7], A[6, 7] = float("inf"), 1.0             # row 7 of the product: infinite, NaN where a zero of B meets it
    B[5, ::9] = 0.0
    A[3, 250] = float("nan")
    B[7, N - 1], B[9, 40] = -float("inf"), 3e38
    A[:, 20], A[11, 20] = 0.0, 3.4e38                # 3.4e38 rounds up to infinity in bf16
    B[11] *= 0.25
    B[9, 40] = 3e38
    A[9, 20] = 0.0
    C = torch.zeros((M, N), device=DEV)
    kf.kfac_profile_gemm(A, B, C, M, N, K, A.shape[1], B.shape[1], N, mode, 0, 0)
    torch.cuda.synchronize()
    a, b = A[:, :M].cpu().numpy().astype(np.float64), B[:, :N].cpu().numpy().astype(np.float64)
    got = C.cpu().numpy().astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = a.T @ b
        mag = np.abs(a).T @ np.abs(b)
        # BLAS may leave NaN out of a sum with zeros: the special rows and columns once more, term by term
        for m in (7, 250):
            ref[m] = (a[:, m:m + 1] * b).sum(axis=0)
        for n in (N - 1,):
            ref[:, n] = (a * b[:, n:n + 1]).sum(axis=0)
    if mode == 2:
        live = np.tril(np.ones((M, N), dtype=bool))
        assert np.all(got[~live] == 0.0)
        ref, mag = np.where(live, -ref, 0.0), np.where(live, mag, 0.0)
    over = np.isfinite(ref) & (mag > 3.4e38)         # a partial sum may leave the range
    assert np.array_equal(np.isnan(got[~over]), np.isnan(ref[~over]))
    inf = np.isinf(ref) & ~over
    assert np.array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref) & ~over
    bound = (3 + K) * 2.0 ** -24 * mag[fin]
    assert np.all(np.abs(got[fin] - ref[fin]) <= bound)
    assert np.isfinite(got[300 % M, :N - 1]).all()


@pytest.mark.parametrize("fill", [float("nan"), 1e30])
def test_columns_between_the_operand_and_its_pitch_have_no_say(fill):
    """Bit for bit the same result whatever lies past the columns of an operand."""
    M, N, K = 257, 513, 200
    A, B = operands(M, N, K, "one_feature", 4)

    def run(x):
        a, b = torch.full((K, 320), x, device=DEV), torch.full((K, 640), x, device=DEV)
        a[:, :M], b[:, :N] = A[:, :M], B[:, :N]
        C = torch.zeros((M, N), device=DEV)
        kf.kfac_profile_gemm(a, b, C, M, N, K, 320, 640, N, 0, 0, 0)
        torch.cuda.synchronize()
        return C
    assert torch.equal(run(fill), run(0.0))


def factor_bound(x, scale):
    """sum over rows of |x_i x_j|, times what the cut and the sums in fp32 may cost per term, and the last bit of the
    smallest fp32 numbers for each of them"""
    mag = np.abs(x).T @ np.abs(x) * scale
    return (4 + x.shape[0]) * (2.0 ** -24 * mag + 2.0 ** -149)


@pytest.mark.parametrize("kind", ["normal", "late", "features", "samples", "two_levels", "tiny"])
@pytest.mark.parametrize("shape", ["rows", "nchw_even", "nchw_odd"])
def test_split_factors(kind, shape):
    """Factors of uneven inputs through the public call, element by element: row-major operands, NCHW operands on maps
    with a multiple of four positions and without, tiles on the diagonal (which share their fragments) and off it."""
    gen = np.random.default_rng(7)
    if shape == "rows":
        B, d_in, d_out, h, w = 700, 513, 256, 1, 1
        d = kf.LayerDesc.linear(d_in - 1, d_out, True, kf.KFAC_F32)
        x = gen.standard_normal((B, d_in - 1))
        y = gen.standard_normal((B, d_out))
    else:
        h, w = (8, 6) if shape == "nchw_even" else (7, 5)
        B, d_in, d_out = 9, 512, 320
        d = kf.LayerDesc.conv2d(d_in, d_out, 1, 1, 0, False, kf.KFAC_F32)
        x = gen.standard_normal((B, d_in, h * w))
        y = gen.standard_normal((B, d_out, h * w))
    for v in (x, y):
        col = np.arange(v.shape[1])
        shp = (1, -1) if v.ndim == 2 else (1, -1, 1)
        if kind == "late":
            v[:len(v) // 2] = 0
        elif kind == "features":
            v *= np.exp(3 * gen.standard_normal(v.shape[1])).reshape(shp)
        elif kind == "samples":
            v *= np.exp(3 * gen.standard_normal(len(v))).reshape((-1,) + (1,) * (v.ndim - 1))
        elif kind == "two_levels":       # columns large in one half of the samples only meet tiny ones of the others
            half = len(v) // 2
            v[:half, col % 2 == 0] *= 1e-12
            v[half:, col % 2 == 1] *= 1e-12
        elif kind == "tiny":             # one column in two next to the smallest fp32 numbers, the others large
            v[:, col % 2 == 0] *= 2.0 ** -119
            v[:, col % 2 == 1] *= 2.0 ** 40
    x, y = x.astype(np.float32), y.astype(np.float32)
    if shape != "rows":
        x, y = x.reshape(B, d_in, h, w), y.reshape(B, d_out, h, w)
    X = x.reshape(B, -1, h * w).transpose(0, 2, 1).reshape(B * h * w, -1).astype(np.float64)
    Y = y.reshape(B, -1, h * w).transpose(0, 2, 1).reshape(B * h * w, -1).astype(np.float64)
    if shape == "rows":
        X = np.concatenate([X, np.ones((B, 1))], axis=1)
    work = torch.empty(kf.kfac_workspace_bytes(d, B, h, w), dtype=torch.uint8, device=DEV)
    A = torch.zeros(X.shape[1], X.shape[1], device=DEV)
    G = torch.zeros(Y.shape[1], Y.shape[1], device=DEV)
    kf.kfac_update_factors(d, torch.from_numpy(x).to(DEV), torch.from_numpy(y).to(DEV), B, h, w, 1.0 / B, 1.0 / B, 0.0, A, G,
                           work)
    torch.cuda.synchronize()
    for got, v in ((A, X), (G, Y)):
        err = np.abs(got.double().cpu().numpy() - v.T @ v / B)
        bound = factor_bound(v, 1.0 / B)
        assert np.all(err <= bound), f"error {np.max(err / np.maximum(bound, 1e-300)):.3f} of the bound"


@pytest.mark.parametrize("shape", ["rows", "nchw_even", "nchw_odd"])
def test_infinite_input_of_a_split_factor(shape):
    """One infinite activation: its row and column of the factor are infinite (NaN where it meets a zero), the rest is
    what it was.  Row-major operands and NCHW ones, whose positions past the end of an image are cut off in the second
    computation of a tile too; tiles on the diagonal and off it."""
    n = 512
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    if shape == "rows":
        B, h, w = 400, 1, 1
        d = kf.LayerDesc.linear(n, 256, False, kf.KFAC_F32)
    else:
        B, (h, w) = 9, (8, 6) if shape == "nchw_even" else (7, 5)
        d = kf.LayerDesc.conv2d(n, 256, 1, 1, 0, False, kf.KFAC_F32)
    X = torch.randn(B * h * w, n, generator=g, device=DEV)            # one row per example and position
    X[17] = X[17].abs() + 0.1
    X[17, 300], X[17, 31] = float("inf"), 0.0
    x = X if shape == "rows" else X.view(B, h, w, n).permute(0, 3, 1, 2).contiguous()
    y = torch.randn((B, 256) if shape == "rows" else (B, 256, h, w), generator=g, device=DEV)
    work = torch.empty(kf.kfac_workspace_bytes(d, B, h, w), dtype=torch.uint8, device=DEV)
    A, G = torch.zeros(n, n, device=DEV), torch.zeros(256, 256, device=DEV)
    kf.kfac_update_factors(d, x, y, B, h, w, 1.0, 1.0, 0.0, A, G, work)
    torch.cuda.synchronize()
    got = A.cpu()
    want = torch.full((n,), float("inf"))
    want[31] = float("nan")
    assert torch.equal(got[300].isnan(), want.isnan()) and torch.equal(got[300].nan_to_num(0.0), want.nan_to_num(0.0))
    assert torch.equal(got[300].isnan(), got[:, 300].isnan())
    keep = torch.arange(n) != 300
    ref = X.double().cpu()[:, keep]
    err = (got[keep][:, keep].double() - ref.T @ ref).abs().numpy()
    assert np.all(err <= factor_bound(ref.numpy(), 1.0))


@pytest.mark.parametrize("sigma", [0.75, 2.0])
def test_preconditioning_of_unevenly_scaled_features(sigma):
    """Features of log-normal scale s: gradients ~ s, inverse ~ 1 / (s s').  Element by element, through the public call."""
    d_in, d_out = 768, 256
    n = d_in + 1
    d = kf.LayerDesc.linear(d_in, d_out, True, kf.KFAC_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(21)
    s = torch.exp(sigma * torch.randn(n, generator=g, device=DEV))
    A = torch.randn(n, n, generator=g, device=DEV) * 0.02
    A = (A + A.T) / 2 + torch.eye(n, device=DEV)
    A = A / s[:, None] / s[None]
    G = torch.randn(d_out, d_out, generator=g, device=DEV) * 0.02
    G = (G + G.T) / 2 + torch.eye(d_out, device=DEV)
    W = torch.randn(d_out, n, generator=g, device=DEV) * s[None]
    work = torch.empty(kf.kfac_workspace_bytes(d, 8, 1, 1), dtype=torch.uint8, device=DEV)
    out = torch.empty(d_out, n, device=DEV)
    kf.kfac_precondition(d, A, G, W, out, work)
    torch.cuda.synchronize()
    a, b, w = A.double().cpu(), G.double().cpu(), W.double().cpu()
    bound = (2 + n + d_out + 4) * 2.0 ** -24 * (b.abs() @ w.abs() @ a.abs())
    worst = ((out.double().cpu() - b @ w @ a).abs() / bound).max().item()
    assert worst <= 1.0, f"error {worst:.3f} of the bound"


@pytest.mark.parametrize("d_in,d_out", [(1023, 400), (1024, 300), (2300, 200), (5000, 130)])
def test_k_slices_of_one_layer(d_in, d_out):
    """A call of one layer: its deep products are cut into slices of 40 stages and more, up to eight of them.  The same
    bound as above, twice: the first product's error passes through the second.  A workspace without room for the slices
    leaves the products in one piece: other bits, or the slices were not used."""
    d = kf.LayerDesc.linear(d_in, d_out, True, kf.KFAC_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    n = d_in + 1
    A, G, W = (torch.randn(*s, generator=g, device=DEV) for s in ((n, n), (d_out, d_out), (d_out, n)))
    A, G = (A + A.T) / 2, (G + G.T) / 2
    work = torch.empty(kf.kfac_workspace_bytes(d, 8, 1, 1), dtype=torch.uint8, device=DEV)
    out = torch.empty(d_out, n, device=DEV)
    kf.kfac_precondition(d, A, G, W, out, work)
    whole = torch.empty_like(out)
    least = (d_out * n * 4 + 255) // 256 * 256
    assert work.numel() > least
    kf.kfac_precondition(d, A, G, W, whole, work[:least])
    torch.cuda.synchronize()
    assert not torch.equal(out, whole), "the slices were not used"
    a, b, w = A.double().cpu(), G.double().cpu(), W.double().cpu()
    mag = b.abs() @ w.abs() @ a.abs()
    bound = (2 + n + d_out + 4) * 2.0 ** -24 * mag
    worst = ((out.double().cpu() - b @ w @ a).abs() / bound).max().item()
    assert worst <= 1.0, f"error {worst:.3f} of the bound"


def test_accuracy_of_a_layer_does_not_depend_on_its_call():
    """Alone in its call a 700 x 500 layer is multiplied by the split kernel, beside many small ones by the fp32 kernels
    (other bits, or the routes were the same): the bound of preconditioning holds for both, and both are equally close."""
    descs = [kf.LayerDesc.linear(699, 500, True, kf.KFAC_F32)] + [kf.LayerDesc.linear(99, 100, True, kf.KFAC_F32)] * 400
    g = torch.Generator(device=DEV)
    g.manual_seed(8)

    def inverse(n):
        r = torch.randn(n, n, generator=g, device=DEV)
        return (r + r.T) * (0.05 / n ** 0.5) + torch.diag(torch.rand(n, generator=g, device=DEV) + 0.5)
    A, G = [inverse(700)] + [inverse(100)] * 400, [inverse(500)] + [inverse(100)] * 400
    W = [torch.randn(500, 700, generator=g, device=DEV)] + [torch.randn(100, 100, generator=g, device=DEV)] * 400
    got = []
    for n in (1, 401):
        one = [1] * n
        work = torch.empty(kf.kfac_workspace_bytes_batched(descs[:n], one, one, one), dtype=torch.uint8, device=DEV)
        out = [torch.empty_like(w) for w in W[:n]]
        kf.kfac_precondition_batched(descs[:n], A[:n], G[:n], W[:n], out, work)
        torch.cuda.synchronize()
        got.append(out[0].double().cpu())
    assert not torch.equal(*got)
    a, b, w = A[0].double().cpu(), G[0].double().cpu(), W[0].double().cpu()
    ref = b @ w @ a
    bound = (2 + 700 + 500 + 4) * 2.0 ** -24 * (b.abs() @ w.abs() @ a.abs())
    for x in got:
        assert ((x - ref).abs() / bound).max().item() <= 1.0
    alone, batched = ((x - ref).norm().item() for x in got)
    assert alone <= 1.1 * batched
