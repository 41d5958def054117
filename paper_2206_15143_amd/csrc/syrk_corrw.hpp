// A factor of a 3x3 / stride 1 / pad 1 fp32 convolution from autocorrelations of its input (syrk_corr3.hpp has the formulas
// and a kernel of its own for 16, 32 and 64 channels on maps it can stage), on the tiles of the split-bf16 kernel.
//
// The input is copied once, channels innermost, every row of the map followed by two zero columns and every image by two
// zero rows: Xp[k][c].  A lag is then a distance in k, whatever its sign along the row, and the zeros make every partner
// outside the map vanish.  The lags of one row distance are neighbours in k, and with a row pitch of C element (k, l C + c)
// of Xp IS element (k + l, c): three plain products A^T B with overlapping rows of A,
//     [3 C, C], [5 C, C], [5 C, C]  =  (Xp from lag (0, 0), (1, -2), (2, -2) on)^T  Xp,
// give all 13 lag matrices, 12.5 C^2 multiply-adds per position of the copy where the patch matrix takes 40.5 per position of
// the map, without the patch matrix (nine times the input) and with slices of 13 C^2 instead of 40.5 C^2 entries to sum.
// The border rows and columns, copied out the same way, give the one-dimensional autocorrelations ([3 C, C] each) and the
// corner pixels their outer products.  K slices are bounded like those of syrk_split.hpp, for the same reason.
// An infinite or NaN input makes every entry of its channel's rows and columns non-finite (a zero of the padding times it
// included), no others.
// Accuracy: an entry of a tap that leaves out a border row or column is the sum over the whole map less the border's, so its
// error is a few 2^-24 of the geometric mean of the two channels' centre-tap entries (which hold every position), where a
// direct sum has the taps' own entries in their place: the same on maps of one scale; on a map whose border is 1000 times
// its inside 4e-7 of the centre taps, and entries of the inside alone have no digits left.  Norm-wise 2.5e-7 on either.
// Small calls keep the patch matrix: corrw_gain in syrk.hip.
// Factor updates in ms, before (patch matrix and split kernel, fused 3x3 kernel up to 64 channels) and now: VGG-16-shaped 2.53
// and 2.02; resnet_cifar of width 20, 24 and 32: 3.65, 6.43, 1.82 and 2.50, 3.12, 1.42; DenseNet-shaped with growth 12 and 24:
// 2.46, 3.07 and 1.86, 1.90; whole updates: ResNet-50-shaped 15.1 and 13.3, DenseNet-201-shaped 19.8 and 15.8.
// Bound: bf16 MFMA (six products each), on small maps the copy's padding: (H + 2)(W + 2) / (H W) = 1.31 at 14 x 14,
// 1.65 at 7 x 7, 2.25 at 4 x 4.
#pragma once

#include "syrk_corr3.hpp"
#include "split_common.hpp"

namespace kfac {

constexpr int kCorrwParts = 512;      // workgroups of the copy per 64 channels aimed for: parts of an image

// Sizes of one factor's workspace, in floats.
struct CorrW {
    int C, H, W, B;
    long PI, Kp, Kr, Kc;              // positions of an image of the copy; rows of K: main, row borders, column borders
    int parts;                        // parts of an image in the copy kernel
    int slices, kper;                 // main products
    int bslices, kper_r, kper_c, kper_q;
    size_t Xp, R, Cc, Q, V, Fp, Bp, Fs, FsT, Bs, BsT, total;      // offsets
    CorrW(int c, int h, int w, int b) : C(c), H(h), W(w), B(b)
    {
        PI = (long)(H + 2) * (W + 2);
        Kp = B * PI;
        Kr = (long)B * (W + 2);
        Kc = (long)B * (H + 2);
        auto cut = [](long k, int n) { return (int)(((k + S_KT - 1) / S_KT + n - 1) / n) * S_KT; };
        const long most = std::max(1l, tuning().split_syrk_max_stages);
        auto stages = [](long k) { return (k + S_KT - 1) / S_KT; };
        slices = (int)((stages(Kp) + most - 1) / most);
        kper = cut(Kp, slices);
        bslices = (int)((stages(std::max(std::max(Kr, Kc), (long)B)) + most - 1) / most);
        kper_r = cut(Kr, bslices);
        kper_c = cut(Kc, bslices);
        kper_q = cut(B, bslices);
        const long groups = (long)B * ((C + 63) / 64), chunks = (PI + 63) / 64;
        parts = (int)std::min(chunks, std::max(1l, kCorrwParts / groups));
        size_t off = 0;
        auto take = [&](size_t n) {
            const size_t o = off;
            off += (n + 63) / 64 * 64;
            return o;
        };
        const size_t cc = (size_t)C * C;
        Xp = take((size_t)Kp * C);
        R = take(2 * (size_t)Kr * C);
        Cc = take(2 * (size_t)Kc * C);
        Q = take(4 * (size_t)B * C);
        V = take((size_t)B * parts * 9 * C);
        Fp = take((size_t)slices * C3_LAGS * cc);
        Bp = take((size_t)bslices * C3_BQ * cc);
        Fs = take(C3_LAGS * cc + C);
        FsT = take(C3_LAGS * cc);
        Bs = take(C3_BQ * cc + (size_t)C3_BV * C);
        BsT = take(C3_BQ * cc);
        total = off;
    }
};

struct CorrWProb {
    const float *x;
    float *Xp, *R, *Cc, *Q, *V, *Fp, *Bp, *Fs, *FsT, *Bs, *BsT;
    int C, H, W, B;
    int parts, slices, bslices;
    int blk_start;
};

struct CorrWTable {
    int count;
    CorrWProb p[kMaxProblems];
};

// The padded, transposed copy, the border rows, columns and corners, and the sums over them all.  A workgroup takes one
// part of one image for 64 channels, 64 positions at a time through LDS: 256 contiguous bytes read along a channel and
// written along a position.
__global__ __launch_bounds__(256) void corrw_copy_kernel(const CorrWTable tab)
{
    __shared__ float t[64][65];
    __shared__ float sums[9][4][64];
    int pi = 0;
    while (pi + 1 < tab.count && (int)blockIdx.x >= tab.p[pi + 1].blk_start) ++pi;
    const CorrWProb &pr = tab.p[pi];
    const int C = pr.C, H = pr.H, W = pr.W, Wp = W + 2;
    const int cb = (C + 63) / 64;
    int local = blockIdx.x - pr.blk_start;
    const int c0 = 64 * (local % cb);
    local /= cb;
    const int part = local % pr.parts, n = local / pr.parts;
    const int PI = (H + 2) * Wp, chunks = (PI + 63) / 64, per = (chunks + pr.parts - 1) / pr.parts;
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int c = c0 + lane;
    float sum[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) sum[q] = 0.f;
    for (int ch = part * per; ch < min(chunks, (part + 1) * per); ++ch) {
        {
            const int p = 64 * ch + lane, a = p / Wp, b = p - a * Wp;
            const bool in = a < H && b < W;
            const float *src = pr.x + (long)n * C * H * W + (in ? a * W + b : 0);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int cc = c0 + g + 4 * i;
                const float v = src[(long)min(cc, C - 1) * H * W];
                t[g + 4 * i][lane] = in ? v : 0.f;
            }
        }
        __syncthreads();
        if (c < C) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int p = 64 * ch + g + 4 * i;
                if (p >= PI) break;
                const int a = p / Wp, b = p - a * Wp;
                const float v = t[lane][g + 4 * i];
                pr.Xp[((long)n * PI + p) * C + c] = v;
                const bool top = a == 0, bottom = a == H - 1, left = b == 0, right = b == W - 1;
                sum[0] += v;
                if (top || bottom) {
                    pr.R[(((long)(bottom ? pr.B : 0) + n) * Wp + b) * C + c] = v;
                    sum[bottom ? 2 : 1] += v;
                }
                if (left || right) {
                    pr.Cc[(((long)(right ? pr.B : 0) + n) * (H + 2) + a) * C + c] = v;
                    sum[right ? 4 : 3] += v;
                    if (top || bottom) {
                        const int q = (bottom ? 2 : 0) + (right ? 1 : 0);
                        pr.Q[((long)q * pr.B + n) * C + c] = v;
#pragma unroll
                        for (int k = 0; k < 4; ++k) sum[5 + k] += k == q ? v : 0.f;
                    }
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) sums[q][g][lane] = sum[q];
    __syncthreads();
    for (int e = threadIdx.x; e < 9 * 64; e += 256) {
        const int q = e >> 6, l = e & 63;
        if (c0 + l < C)
            pr.V[(((long)n * pr.parts + part) * 9 + q) * C + c0 + l] = (sums[q][0][l] + sums[q][1][l]) + (sums[q][2][l] + sums[q][3][l]);
    }
}

// Sums over the slices, fixed order: the matrices as the products leave them ([partner][channel]) and, through LDS,
// transposed; the vectors.  A workgroup per 32 x 32 tile of a matrix, then one per 256 entries of the vectors.
__global__ __launch_bounds__(256) void corrw_sum_kernel(const CorrWTable tab)
{
    __shared__ float t[32][33];
    int pi = 0;
    while (pi + 1 < tab.count && (int)blockIdx.x >= tab.p[pi + 1].blk_start) ++pi;
    const CorrWProb &pr = tab.p[pi];
    const int C = pr.C, side = (C + 31) / 32, tid = threadIdx.x;
    const long cc = (long)C * C;
    int local = blockIdx.x - pr.blk_start;
    const int mats = (C3_LAGS + C3_BQ) * side * side;
    if (local >= mats) {
        const int e = (local - mats) * 256 + tid;
        if (e >= 9 * C) return;
        const int q = e / C, c = e - q * C, n = pr.B * pr.parts;
        const float *src = pr.V + (long)q * C + c;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        int i = 0;
        for (; i + 4 <= n; i += 4)
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] += src[(long)(i + k) * 9 * C];
        for (; i < n; ++i) s[0] += src[(long)i * 9 * C];
        const float v = (s[0] + s[1]) + (s[2] + s[3]);
        if (q == 0) pr.Fs[C3_LAGS * cc + c] = v;
        else pr.Bs[C3_BQ * cc + (long)(q - 1) * C + c] = v;
        return;
    }
    const int m = local / (side * side);
    local -= m * side * side;
    const int r0 = 32 * (local / side), q0 = 32 * (local % side);
    const bool lag = m < C3_LAGS;
    const int parts = lag ? pr.slices : pr.bslices;
    // A matrix of lag zero (and a corner's) is symmetric, but the split product of (c, c') and of (c', c) adds the same terms
    // in another order: the tiles on and below its diagonal stand for both, so that the factor is symmetric to the bit.
    const int bm = m - C3_LAGS;
    const bool self = lag ? m == 0 : (bm >= 12 || bm % 3 == 0);
    if (self && r0 < q0) return;
    const long stride = (lag ? C3_LAGS : C3_BQ) * cc, base = (lag ? m : m - C3_LAGS) * cc;
    const float *src = (lag ? pr.Fp : pr.Bp) + base;
    const int r = tid >> 3, c4 = (tid & 7) * 4;
    floatx4 a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (r0 + r < C && q0 + c4 < C) {                  // (C is a multiple of 4)
        const float *e = src + (long)(r0 + r) * C + q0 + c4;
        int p = 0;
        for (; p + 4 <= parts; p += 4)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] += *reinterpret_cast<const floatx4 *>(e + (p + k) * stride);
        for (; p < parts; ++p) a[0] += *reinterpret_cast<const floatx4 *>(e + p * stride);
    }
    floatx4 v = (a[0] + a[1]) + (a[2] + a[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) t[r][c4 + k] = v[k];
    __syncthreads();
    floatx4 w;
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = t[c4 + k][r];
    if (self && r0 == q0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = w[k] = c4 + k > r ? w[k] : v[k];
    }
    float *direct = (lag ? pr.FsT : pr.BsT) + base, *mirror = (lag ? pr.Fs : pr.Bs) + base;
    if (r0 + r < C && q0 + c4 < C) {
        *reinterpret_cast<floatx4 *>(direct + (long)(r0 + r) * C + q0 + c4) = v;
        if (self) *reinterpret_cast<floatx4 *>(mirror + (long)(r0 + r) * C + q0 + c4) = v;
    }
    if (q0 + r < C && r0 + c4 < C && !(self && r0 == q0)) {
        *reinterpret_cast<floatx4 *>(mirror + (long)(q0 + r) * C + r0 + c4) = w;
        if (self) *reinterpret_cast<floatx4 *>(direct + (long)(q0 + r) * C + r0 + c4) = w;
    }
}

}  // namespace kfac
