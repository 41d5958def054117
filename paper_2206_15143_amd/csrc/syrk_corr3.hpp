// A factor of a 3x3 / stride 1 / pad 1 convolution from spatial autocorrelations of its input.
//
// With zero padding, entry ((c,i,j), (c',i',j')) of  A = sum over patches of  a a^T  (Eq. 4 of the DP-KFAC
// paper, the convolution seen as a linear map over patches) is
//     sum_n sum_{a in Ra(i)} sum_{b in Rb(j)}  x[n,c,a,b] * x[n,c',a+di,b+dj],      (di, dj) = (i'-i, j'-j),
// where x is 0 outside the image and Ra(0) = [0,H-2], Ra(1) = [0,H-1], Ra(2) = [1,H-1] (likewise Rb).  The sum
// over ALL (a,b) depends on (di,dj) only: the autocorrelation F(di,dj)[c][c'] of the input at one of 25 lags,
// of which 13 are independent (F(-d)[c][c'] = F(d)[c'][c]).  What the window removes is a single image row
// (for i = 0 or 2) and/or a single column (j = 0 or 2), and such a term is non-zero only when the partner
// lands in the same row (i' = i) resp. column (j' = j):
//     A = F(d) - [i'=i in {0,2}] Row(a*, dj) - [j'=j in {0,2}] Col(b*, di) + [both] Corner(a*, b*),
// with a* = H-1 for i = 0 and 0 for i = 2 (b* likewise), Row / Col the 1-D autocorrelations of that border
// row / column and Corner the outer product of the corner pixel.  The bias border (column sums of the patch
// matrix) follows the same inclusion-exclusion on plain sums.  The result is the same matrix as the direct
// sum (up to rounding order) for 13 instead of 45 MFMA tiles per 16 x 16 channel pair and k-step.  The subtraction leaves
// errors relative to the centre-tap entries of the two channels (see syrk_corrw.hpp).
//
// Three steps: corr3_main_kernel (the 13 lag matrices, split over images, on the MFMA units),
// corr3_border_kernel (rows, columns, corners; MFMA as well, K = border pixels), corr3_sum_kernel +
// corr3_assemble_kernel (sum of the splits, assembly of A with scale and running average, both triangles).
#pragma once

#include "common.hpp"
#include "split_common.hpp"
#include "tn_engine.hpp"
#include "wave_common.hpp"

namespace kfac {

constexpr int C3_LAGS = 13;
constexpr int C3_BQ = 16;          // border matrices per layer: 6 row, 6 column, 4 corner
constexpr int C3_BV = 8;           // border vectors per layer: 2 row sums, 2 column sums, 4 corner sums
constexpr int C3_CHUNKS = 5;       // image chunks of the border kernels (5 x 4 pair groups x 36 layers = 720 workgroups at 64 channels: under 3 per CU)

struct CorrProb {
    const float *x;    // NCHW input [B, C, H, W]
    float *Fp;         // [parts][13][C][C] lag matrices per part, then [parts][C] channel sums per part
    float *Fs;         // [13][C][C] + [C]: summed over the parts
    float *Bp;         // [chunks][16][C][C], then [chunks][8][C]
    float *Bs;         // [16][C][C] + [8][C]: summed over the chunks
    float *FsT, *BsT;  // the matrices of Fs and Bs transposed ([l][c'][c]): the assembly reads both orders along rows
    float *cols;       // [B][2][C][H]: first and last image column, written by the main kernel for the border kernel
    float *F;          // factor [dF, dF], dF = 9 C + has_bias
    int C, H, W, B;
    int SR, strips;    // rows per strip, strips per image
    int units;         // B * strips
    int upb;           // units per block of the main kernel
    int parts;         // blocks (ranges of units) of the main kernel
    int fblocks;       // blocks of the sum kernel for the lag matrices
    int plane;         // octets per channel plane of a slab
    int blk_start;     // first block of this problem in the kernel at hand
    int has_bias;
    float scale, decay;
};

struct CorrTable {
    int count;
    int starts[kMaxProblems];     // blk_start of every problem, compact: searched by bisection
    CorrProb p[kMaxProblems];
};

__device__ __forceinline__ int corr_locate(const CorrTable &tab, int blk)
{
    int lo = 0, hi = tab.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (blk >= tab.starts[mid]) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------------------------------------
// Lag matrices, on the bf16 units at fp32 accuracy (split_common.hpp: every value cut into three pieces, six products).
// A workgroup (eight product and four staging wavefronts, one per CU) walks (image, strip) units: the strip of all C channels with two
// halo rows below lies in LDS as octets, eight pixels of a row and channel in three pieces of 16 bytes (double buffered; the
// loads of the next unit are in flight under the products, and the staging wavefronts cut and store it beside them).
// A k-step is four octets, one per 16 lanes.  The sum over a row of x[c][a] x'[c'][a + dj] is taken as that of x[c][y - dj]
// x'[c'][y]: the shift is applied to the A operand alone, in registers, from the octet and the pixel pairs beside it, so that
// five shifts of A serve the three row lags of B, and all operands are aligned 16-byte reads.
//   NT = 1 (C = 16): one tile pair; the product wavefronts take every eighth k-step.
//   NT = 2 (C = 32): four tile pairs, each by two wavefronts with every second k-step.
//   NT = 4 (C = 64): 16 tile pairs, half of them (two B tiles) in either of two workgroups that share a range of units.
// Bound: MFMA, 78 of 16 cycles per k-step and wavefront, with 115 VALU operations and 16 operand reads beside them.  36 layers
// of 16 x 32 x 32, batch 128: 159 us, 1185 TFLOP/s of bf16 products (the library's large split product runs at 1320, short of
// power); 32 x 16 x 16: 147, 64 x 8 x 8: 154.  On the fp32 MFMA, at 120 of its 157 TFLOP/s: 261, 260 and 277 us.  The six products
// interleaved by hand with the shifts and sums of their neighbours: no gain.  Six wavefronts a workgroup, two of them on a
// CU, do not run together (their wavefronts 0 and 1 want the same SIMDs): 219, 175, 203 us.
// A wavefront with a result that is not finite (inf or NaN in the input, values from 2^112 on) computes its tiles once
// more on the fp32 MFMA from the input in memory, which leaves what fp32 arithmetic gives.
constexpr int C3_PW = 8, C3_SW = 4;              // product and staging wavefronts: three a SIMD, of 168 registers
constexpr int C3_THREADS = 64 * (C3_PW + C3_SW);
constexpr int C3_ITEMS = 6;                      // octets per staging thread and slab at most (checked by the planner)
constexpr int C3_OCT = 48;                       // bytes of an octet
constexpr int C3_ZERO = 64;                      // bytes ahead of the slabs: an octet of zeros
constexpr int corr3_ks(int C) { return C == 16 ? 8 : C == 32 ? 2 : 1; }       // product wavefronts that split the k-steps
constexpr int corr3_rounds(int C) { return C == 16 ? 3 : C == 32 ? 1 : 0; }     // of the sum over them (log2)
constexpr int C3_RED = 8192;                     // bytes of LDS for the channel sums, ahead of four wavefronts' lag tiles
constexpr int corr3_tail_lds(int C) { return C3_RED + (corr3_ks(C) > 1 ? 4 * C3_LAGS * 64 * 16 : 0); }
constexpr int corr3_sharers(int C) { return C == 64 ? 2 : 1; }  // workgroups that share a range of units
constexpr __host__ __device__ int corr3_lag(int di, int dj) { return 5 * di + dj; }      // di = 0: dj = 0, 1, 2; else -2 .. 2

template <int NT>
__global__ __launch_bounds__(C3_THREADS, 3) void corr3_main_kernel(const CorrTable tab)
{
    extern __shared__ __align__(16) unsigned char corr_lds[];
    constexpr int C = 16 * NT, KS = corr3_ks(C), SHARERS = corr3_sharers(C);
    const CorrProb &pr = tab.p[corr_locate(tab, blockIdx.x)];
    const int blk_raw = blockIdx.x - pr.blk_start;
    const int blk = blk_raw / SHARERS, share = blk_raw - blk * SHARERS;
    const int u0 = blk * pr.upb, u1 = min(pr.units, u0 + pr.upb);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int H = pr.H, W = pr.W, SR = pr.SR, plane = pr.plane;
    const int opr = (W + 7) >> 3;                          // octets per image row
    const unsigned slab = (unsigned)(C * plane * C3_OCT);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.x), 0,
                                                                        (int)((long)pr.B * C * H * W * 4), 0x00020000);   // below 2^31 (planner)

    // Wavefronts 8 .. 11 stage the slabs.  One barrier per unit: past barrier `it` the slab of unit `it` is complete and every
    // product wavefront is done with unit it - 1, whose buffer is then filled with unit it + 1.
    if (w >= C3_PW) {
        const int tid = threadIdx.x - 64 * C3_PW, rows = SR + 2, per_c = rows * opr, nitems = C * per_c;
        unsigned vo[C3_ITEMS];                             // byte offset of the octet in the image, from row a0 on
        int vr[C3_ITEMS];                                  // its row of the slab
        unsigned at[C3_ITEMS], co[C3_ITEMS];               // its place in a slab, and that of its row among the border columns
        unsigned first = 0, last = 0;                      // bit per octet: it is the first, the last of its image row
        float sums[C3_ITEMS];
        floatx4 raw[2][C3_ITEMS][2];                       // the loads of two units in flight
#pragma unroll
        for (int j = 0; j < C3_ITEMS; ++j) {
            const int q = tid + 64 * C3_SW * j, c = q / per_c, rem = q - c * per_c, r = rem / opr;
            vr[j] = q < nitems ? r : 1 << 20;
            vo[j] = (unsigned)(((c * H + r) * W + 8 * (rem - r * opr)) * 4);
            at[j] = C3_ZERO + (unsigned)((c * plane + rem) * C3_OCT);
            co[j] = (unsigned)(c * H + r);
            first |= (rem == r * opr ? 1u : 0u) << j;
            last |= (rem == r * opr + opr - 1 ? 1u : 0u) << j;
            sums[j] = 0.f;
        }
        if (tid < C3_ZERO / 4) reinterpret_cast<float *>(corr_lds)[tid] = 0.f;
        auto load = [&](int u, floatx4 (&x)[C3_ITEMS][2]) {        // past the last unit: nothing is read
            const int n = u / pr.strips, a0 = (u - n * pr.strips) * SR;
            const unsigned so = (unsigned)((n * C * H + a0) * W) * 4u;
#pragma unroll
            for (int j = 0; j < C3_ITEMS; ++j) {
                const bool in = u < u1 && a0 + vr[j] < H;
                const bool half = (W & 4) && (last >> j & 1);      // four of its pixels lie past the row
                x[j][0] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? vo[j] : W_OOB, so, 0));
                x[j][1] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rx, in && !half ? vo[j] + 16u : W_OOB, so, 0));
            }
        };
        auto store = [&](int u, const floatx4 (&x)[C3_ITEMS][2], int buf) {
            const int n = u / pr.strips, a0 = (u - n * pr.strips) * SR;
#pragma unroll
            for (int j = 0; j < C3_ITEMS; ++j) {
                if (64 * C3_SW * j >= nitems) continue;    // uniform
                if (vr[j] >= rows) continue;
                float x0[4], x1[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { x0[e] = x[j][0][e]; x1[e] = x[j][1][e]; }
                if (vr[j] < SR) {
                    sums[j] += ((x0[0] + x0[1]) + (x0[2] + x0[3])) + ((x1[0] + x1[1]) + (x1[2] + x1[3]));
                    // the first and the last pixel of every image row also go to a compact buffer (the border kernel would
                    // otherwise pull a whole cache line per pixel; 64 channels have short columns, read from the input)
                    if (NT != 4 && a0 + vr[j] < H) {
                        float *cols = pr.cols + (long)n * 2 * C * H + a0;
                        if (first >> j & 1) cols[co[j]] = x0[0];
                        if (last >> j & 1) cols[co[j] + (unsigned)(C * H)] = (W & 4) ? x0[3] : x1[3];
                    }
                }
                SplitCut k0, k1;
                suint4 *to = reinterpret_cast<suint4 *>(corr_lds + at[j] + (unsigned)buf * slab);
                k0.scale(x0); k1.scale(x1);
#pragma unroll
                for (int piece = 0; piece < 2; ++piece) {
                    k0.half(x0, 0, 4); k1.half(x1, 0, 4);
                    const suint2 p = k0.pack(), r = k1.pack();
                    to[piece] = suint4{p.x, p.y, r.x, r.y};
                    k0.top(0, 4); k1.top(0, 4);
                    k0.rest(x0, 0, 4); k1.rest(x1, 0, 4);
                }
                const suint2 p = k0.pack_last(x0), r = k1.pack_last(x1);
                to[2] = suint4{p.x, p.y, r.x, r.y};
            }
        };
        load(u0, raw[0]);
        __builtin_amdgcn_sched_barrier(0);
        load(u0 + 1, raw[1]);
        for (int u = u0; u < u1; u += 2) {                 // (no condition on the loads: their number is what the waits count)
            store(u, raw[0], 0);
            __builtin_amdgcn_sched_barrier(0);
            load(u + 2, raw[0]);
            __syncthreads();
            if (u + 1 >= u1) break;
            store(u + 1, raw[1], 1);
            __builtin_amdgcn_sched_barrier(0);
            load(u + 3, raw[1]);
            __syncthreads();
        }
        // channel sums: the octets of a channel in order
        __syncthreads();
        float *red = reinterpret_cast<float *>(corr_lds);
#pragma unroll
        for (int j = 0; j < C3_ITEMS; ++j)
            if (tid + 64 * C3_SW * j < nitems) red[tid + 64 * C3_SW * j] = sums[j];
        static_assert(C3_ITEMS * 64 * C3_SW * 4 <= C3_RED, "the channel sums fit");
        __syncthreads();
        if (share == 0 && tid < C) {
            float t = 0.f;
            for (int o = 0; o < SR * opr; ++o) t += red[tid * per_c + o];
            pr.Fp[(long)pr.parts * (C3_LAGS * C * C) + (long)blk * C + tid] = t;
        }
        for (int r = 1; r < corr3_rounds(C); ++r) __syncthreads();
        return;
    }

    const int lr = lane & 15, kk = lane >> 4;
    const int ct = NT == 1 ? 0 : NT == 2 ? (w >> 1) & 1 : w & 3;
    const int ctp = NT == 1 ? 0 : NT == 2 ? w & 1 : 2 * share + (w >> 2);
    floatx4 acc[C3_LAGS];
#pragma unroll
    for (int l = 0; l < C3_LAGS; ++l) acc[l] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int noct = SR * opr;                                 // octets of a strip
    const int gfirst = NT == 1 ? w : NT == 2 ? w >> 2 : 0;
    const int nsteps = ((noct + 3) / 4 - gfirst + KS - 1) / KS;
    const int dcol = (4 * KS) % opr;
    for (int u = u0, it = 0; u < u1; ++u, ++it) {
        __syncthreads();
        const unsigned b0 = C3_ZERO + (unsigned)(it & 1) * slab;
        const unsigned pa = b0 + (unsigned)((16 * ct + lr) * plane * C3_OCT);
        const unsigned pb = b0 + (unsigned)((16 * ctp + lr) * plane * C3_OCT);
        int o = 4 * gfirst + kk, col = o % opr;
        for (int s = 0; s < nsteps; ++s) {
            const bool live = o < noct;
            const unsigned oa = live ? pa + (unsigned)(o * C3_OCT) : 0u;
            const unsigned op = live && col > 0 ? oa - C3_OCT + 12u : 0u;          // the pixel pairs beside the octet
            const unsigned on = live && col + 1 < opr ? oa + C3_OCT : 0u;
            const unsigned ob = pb + (unsigned)((live ? o : 0) * C3_OCT);
            suint4 m[3], b[3][3];
            unsigned p[3], n[3];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                m[e] = *reinterpret_cast<const suint4 *>(corr_lds + oa + 16 * e);
                p[e] = *reinterpret_cast<const unsigned *>(corr_lds + op + 16 * e);
                n[e] = *reinterpret_cast<const unsigned *>(corr_lds + on + 16 * e);
            }
#pragma unroll
            for (int di = 0; di < 3; ++di)
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    b[di][e] = *reinterpret_cast<const suint4 *>(corr_lds + ob + (unsigned)(di * opr * C3_OCT) + 16 * e);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                constexpr int order[5] = {0, 1, 2, -1, -2};
                const int dj = order[k];
                suint4 f[3];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const suint4 q = m[e];
                    if (dj == 0) f[e] = q;
                    else if (dj == 2) f[e] = suint4{p[e], q.x, q.y, q.z};
                    else if (dj == -2) f[e] = suint4{q.y, q.z, q.w, n[e]};
                    else if (dj == 1)
                        f[e] = suint4{__builtin_amdgcn_alignbit(q.x, p[e], 16), __builtin_amdgcn_alignbit(q.y, q.x, 16),
                                      __builtin_amdgcn_alignbit(q.z, q.y, 16), __builtin_amdgcn_alignbit(q.w, q.z, 16)};
                    else
                        f[e] = suint4{__builtin_amdgcn_alignbit(q.y, q.x, 16), __builtin_amdgcn_alignbit(q.z, q.y, 16),
                                      __builtin_amdgcn_alignbit(q.w, q.z, 16), __builtin_amdgcn_alignbit(n[e], q.w, 16)};
                }
                // The MFMA cuts off the low bits of what it adds to an accumulator: the six products of a k-step are summed from
                // zero, smallest first, and added to the running sum with round-to-nearest.  (One chain over 64 k-steps: error
                // of the factor 1.3e-6 on zero-mean data; this way 5e-8, and 1.1e-7 on the fp32 MFMA.)
                constexpr int fa[6] = {1, 0, 2, 0, 1, 0}, fb[6] = {1, 2, 0, 1, 0, 0};
                floatx4 sum[3] = {};
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int di = dj < 0 ? 1 : 0; di < 3; ++di)
                        sum[di] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(sbf16x8, f[fa[t]]), __builtin_bit_cast(sbf16x8, b[di][fb[t]]), sum[di], 0, 0, 0);
#pragma unroll
                for (int di = dj < 0 ? 1 : 0; di < 3; ++di) acc[corr3_lag(di, dj)] += sum[di];
            }
            o += 4 * KS;
            col += dcol;
            col -= col >= opr ? opr : 0;
        }
    }
    bool bad = false;
#pragma unroll
    for (int l = 0; l < C3_LAGS; ++l)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            bad |= !(fabsf(acc[l][v]) < __builtin_inff());
            acc[l][v] *= kSplitUnscale;
        }
    if (__any(bad)) {
#pragma unroll
        for (int l = 0; l < C3_LAGS; ++l) acc[l] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int ca = 16 * ct + lr, cb = 16 * ctp + lr;
        for (int u = u0; u < u1; ++u) {
            const int img = u / pr.strips, a0 = (u - img * pr.strips) * SR;
            const unsigned so = (unsigned)(img * C * H * W) * 4u;
            auto pixel = [&](int c, int row, int x) {
                return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    rx, row < H && x >= 0 && x < W ? (unsigned)(((c * H + row) * W + x) * 4) : W_OOB, so, 0));
            };
            for (int s = 0; s < nsteps; ++s)
                for (int o = 4 * (gfirst + s * KS); o < min(noct, 4 * (gfirst + s * KS) + 4); ++o) {
                    const int row = a0 + o / opr, y0 = 8 * (o % opr) + kk;
                    for (int y = y0; y < y0 + 8; y += 4) {
                        float a[5], b[3];
#pragma unroll
                        for (int k = 0; k < 5; ++k) a[k] = pixel(ca, row, y - (k - 2));
#pragma unroll
                        for (int di = 0; di < 3; ++di) b[di] = pixel(cb, row + di, y);
#pragma unroll
                        for (int di = 0; di < 3; ++di)
#pragma unroll
                            for (int dj = di ? -2 : 0; dj < 3; ++dj)
                                acc[corr3_lag(di, dj)] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[dj + 2], b[di], acc[corr3_lag(di, dj)], 0, 0, 0);
                    }
                }
        }
    }
    // sum over the wavefronts that split the k-steps, halving their number: the upper half leaves its tiles in LDS, the lower
    // half adds them to its own (every place is read by the wavefront that writes it in the next round)
    __syncthreads();       // the slabs are free, here and for the channel sums
    int half = 4;
    auto place = [&](int slot, int l) -> floatx4 & {
        return *reinterpret_cast<floatx4 *>(corr_lds + C3_RED + (unsigned)(((slot * C3_LAGS + l) * 64 + lane) * 16));
    };
#pragma unroll
    for (int r = 0; r < (KS > 1 ? corr3_rounds(C) : 1); ++r) {
        if (KS > 1 && w >= half && w < 2 * half)
#pragma unroll
            for (int l = 0; l < C3_LAGS; ++l) place(w & 3, l) = acc[l];
        __syncthreads();
        if (KS > 1 && w < half)
#pragma unroll
            for (int l = 0; l < C3_LAGS; ++l) acc[l] += place((w + half) & 3, l);
        half >>= 1;
    }
    if (KS > 1 && gfirst != 0) return;
    float *Fo = pr.Fp + (long)blk * (C3_LAGS * C * C);
#pragma unroll
    for (int l = 0; l < C3_LAGS; ++l)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            Fo[(l * C + 16 * ct + 4 * kk + v) * C + 16 * ctp + lr] = acc[l][v];
}

// ---------------------------------------------------------------------------------------------------------
// Border terms.  One workgroup per (layer, side, image chunk); side 0 / 1 = image row 0 / H-1, 2 / 3 = column
// 0 / W-1, 4 = the four corners.  For a row or column: per image the line [C][L] (+2 zero cells) is staged in
// LDS, a k-step is four consecutive pixels of the line, lags 0, 1, 2.  Corners: the "line" of a corner is its
// value in the images of the chunk (k runs over images), lag 0 only.
// Wavefront w takes the channel-tile pairs w, w + 4, ...
template <int NT>
__global__ __launch_bounds__(256) void corr3_border_kernel(const CorrTable tab)
{
    constexpr int C = 16 * NT;
    constexpr int NP = NT * NT;                       // tile pairs
    constexpr int PPW = (NP + 3) / 4;                 // pairs per wavefront
    constexpr int LMAX = 64 + 4;
    __shared__ float line[C * LMAX];

    const CorrProb &pr = tab.p[corr_locate(tab, blockIdx.x)];
    const int local = blockIdx.x - pr.blk_start;
    const int side = local / C3_CHUNKS, ch = local - side * C3_CHUNKS;
    const int per = (pr.B + C3_CHUNKS - 1) / C3_CHUNKS;
    const int n0 = ch * per, n1 = min(pr.B, n0 + per);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int lr = lane & 15, kk = lane >> 4;
    const int H = pr.H, W = pr.W;
    float *Bm = pr.Bp + (long)ch * (C3_BQ * C * C);
    float *Bv = pr.Bp + (long)C3_CHUNKS * (C3_BQ * C * C) + (long)ch * (C3_BV * C);

    if (side < 4) {
        const bool is_row = side < 2;
        const int L = is_row ? W : H;                 // line length (a multiple of 4 for rows; any for columns)
        const int fixed = (side & 1) ? (is_row ? H - 1 : W - 1) : 0;
        for (int i = tid; i < C * LMAX; i += 256) line[i] = 0.f;
        floatx4 acc[PPW][3];
#pragma unroll
        for (int p = 0; p < PPW; ++p)
#pragma unroll
            for (int l = 0; l < 3; ++l) acc[p][l] = floatx4{0.f, 0.f, 0.f, 0.f};
        float vs[PPW];
#pragma unroll
        for (int p = 0; p < PPW; ++p) vs[p] = 0.f;
        const int nks = (L + 3) / 4;
        // the elements of the line this thread moves (same for every image): global offset inside an image, LDS index
        constexpr int EPT = (C * 64 + 255) / 256;
        int goff[EPT], loff[EPT];
        constexpr int DEPTH = 4;                              // images whose loads are in flight
        float nxt[DEPTH][EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int i = tid + 256 * k;
            goff[k] = -1;
            loff[k] = 0;
            if (i < C * L) {
                const int c = i / L, p = i - c * L;
                goff[k] = is_row ? (c * H + fixed) * W + p
                                 : (NT == 4 ? (c * H + p) * W + fixed : ((side & 1) * C + c) * H + p);   // columns: compact buffer below 64 channels
                loff[k] = c * LMAX + p;
            }
        }
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            if (n0 + j < n1) {
                const float *img = (is_row || NT == 4) ? pr.x + (long)(n0 + j) * C * H * W : pr.cols + (long)(n0 + j) * 2 * C * H;
#pragma unroll
                for (int k = 0; k < EPT; ++k) nxt[j][k] = goff[k] >= 0 ? img[goff[k]] : 0.f;
            }
        }
        for (int nb = n0; nb < n1; nb += DEPTH) {
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                const int n = nb + j;
                if (n >= n1) break;
                __syncthreads();                              // the products on the previous line are done
#pragma unroll
                for (int k = 0; k < EPT; ++k)
                    if (goff[k] >= 0) line[loff[k]] = nxt[j][k];
                __syncthreads();
                if (n + DEPTH < n1) {                         // refill this register set: in flight for DEPTH lines
                    const float *img = (is_row || NT == 4) ? pr.x + (long)(n + DEPTH) * C * H * W
                                                            : pr.cols + (long)(n + DEPTH) * 2 * C * H;
#pragma unroll
                    for (int k = 0; k < EPT; ++k) nxt[j][k] = goff[k] >= 0 ? img[goff[k]] : 0.f;
                }
#pragma unroll
                for (int p = 0; p < PPW; ++p) {
                    const int pair = w + 4 * p;
                    if (pair >= NP) continue;
                    const int ct = pair / NT, ctp = pair - ct * NT;
                    const float *pa = line + (16 * ct + lr) * LMAX + kk;
                    const float *pb = line + (16 * ctp + lr) * LMAX + kk;
                    for (int ks = 0; ks < nks; ++ks) {
                        const float a = pa[4 * ks];
                        if (ctp == 0) vs[p] += a;
#pragma unroll
                        for (int l = 0; l < 3; ++l)
                            acc[p][l] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, pb[4 * ks + l], acc[p][l], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PPW; ++p) {
            const int pair = w + 4 * p;
            if (pair >= NP) continue;
            const int ct = pair / NT, ctp = pair - ct * NT;
#pragma unroll
            for (int l = 0; l < 3; ++l)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    Bm[((3 * side + l) * C + 16 * ct + 4 * kk + v) * C + 16 * ctp + lr] = acc[p][l][v];
            float s = vs[p];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (ctp == 0 && kk == 0) Bv[side * C + 16 * ct + lr] = s;
        }
    } else {
        // corners: line[q][c][k] = value of corner q of channel c in image n0 + k
        const int nimg = n1 - n0;                     // at most LMAX - 4 (checked by the planner)
        floatx4 acc[PPW][4];
#pragma unroll
        for (int p = 0; p < PPW; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[p][q] = floatx4{0.f, 0.f, 0.f, 0.f};
        float vs[PPW][4];
#pragma unroll
        for (int p = 0; p < PPW; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) vs[p][q] = 0.f;
        const int nks = (nimg + 3) / 4;
        for (int q = 0; q < 4; ++q) {
            const int a = (q & 2) ? H - 1 : 0, b = (q & 1) ? W - 1 : 0;
            // one cache line per value: all loads of a thread in flight before the first is stored
            constexpr int EPC = (C * LMAX + 255) / 256;
            float val[EPC];
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const int i = tid + 256 * e;
                const int c = i / LMAX, k = i - c * LMAX;
                const bool ok = i < C * LMAX && k < nimg;
                const float v = pr.x[ok ? (((long)(n0 + k) * C + c) * H + a) * W + b : 0];
                val[e] = ok ? v : 0.f;
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const int i = tid + 256 * e;
                if (i < C * LMAX) line[i] = val[e];
            }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < PPW; ++p) {
                const int pair = w + 4 * p;
                if (pair >= NP) continue;
                const int ct = pair / NT, ctp = pair - ct * NT;
                const float *pa = line + (16 * ct + lr) * LMAX + kk;
                const float *pb = line + (16 * ctp + lr) * LMAX + kk;
                for (int ks = 0; ks < nks; ++ks) {
                    const float av = pa[4 * ks];
                    if (ctp == 0) vs[p][q] += av;
                    acc[p][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, pb[4 * ks], acc[p][q], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PPW; ++p) {
            const int pair = w + 4 * p;
            if (pair >= NP) continue;
            const int ct = pair / NT, ctp = pair - ct * NT;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    Bm[((12 + q) * C + 16 * ct + 4 * kk + v) * C + 16 * ctp + lr] = acc[p][q][v];
                float s = vs[p][q];
                s += __shfl_xor(s, 16);
                s += __shfl_xor(s, 32);
                if (ctp == 0 && kk == 0) Bv[(4 + q) * C + 16 * ct + lr] = s;
            }
        }
    }
}

// Border terms of small maps (H * W <= 64, 32 or 64 channels), where rows, columns and corners together are a
// large part of every plane and gathering them side by side pulls the input several times over: a workgroup
// stages whole images (contiguous, read once per group of channel-tile pairs) and takes all sixteen border
// matrices from LDS.  One workgroup per (layer, image chunk, group of four tile pairs), one pair per wavefront;
// the loads of two images are in flight.
// Cells past the end of a line are masked in the operand, not padded.
template <int NT>
__global__ __launch_bounds__(256) void corr3_border_plane_kernel(const CorrTable tab)
{
    constexpr int C = 16 * NT;
    constexpr int NG = NT * NT / 4;                   // groups of four tile pairs
    constexpr int PL = 64 + 4;                        // cells per channel plane in LDS
    constexpr int DEPTH = 2;                          // images whose loads are in flight (more would cost a wavefront per SIMD)
    __shared__ __align__(16) float img[C * PL];

    const CorrProb &pr = tab.p[corr_locate(tab, blockIdx.x)];
    const int local = blockIdx.x - pr.blk_start;
    const int ch = local / NG, pg = local - ch * NG;
    const int per = (pr.B + C3_CHUNKS - 1) / C3_CHUNKS;
    const int n0 = ch * per, n1 = min(pr.B, n0 + per);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, kk = lane >> 4;
    const int H = pr.H, W = pr.W, HW = H * W;
    const int pair = 4 * pg + w, ct = pair / NT, ctp = pair - ct * NT;
    float *Bm = pr.Bp + (long)ch * (C3_BQ * C * C);
    float *Bv = pr.Bp + (long)C3_CHUNKS * (C3_BQ * C * C) + (long)ch * (C3_BV * C);

    // what this thread moves per image: float4 f of the image -> plane c, cell p
    int gofs[NT], lofs[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int e = 4 * (tid + 256 * k);
        gofs[k] = -1;
        lofs[k] = 0;
        if (e < C * HW) {
            const int c = e / HW;
            gofs[k] = e;
            lofs[k] = c * PL + (e - c * HW);
        }
    }
    floatx4 regs[DEPTH][NT];
    auto fetch = [&](int j, int n) {
        const float *src = pr.x + (long)n * C * HW;
#pragma unroll
        for (int k = 0; k < NT; ++k) regs[j][k] = *reinterpret_cast<const floatx4 *>(src + (gofs[k] >= 0 ? gofs[k] : 0));
    };
    // matrices: 3 * side + lag for the sides row 0, row H-1, column 0, column W-1, then the four corners;
    // vectors: the four sides, then the four corners
    floatx4 acc[C3_BQ];
    float vs[C3_BV];
#pragma unroll
    for (int m = 0; m < C3_BQ; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < C3_BV; ++m) vs[m] = 0.f;
    const float *pa = img + (16 * ct + lr) * PL;
    const float *pb = img + (16 * ctp + lr) * PL;

    // one k-step of the two sides of a direction: position p = 4 ks + kk of the line, cells org + p * step
    auto lines = [&](int L, int step, int org1, int m0, int v0) {
        const int nks = (L + 3) / 4;
#pragma unroll 2
        for (int ks = 0; ks < nks; ++ks) {
            const int p = 4 * ks + kk;
            const int c0 = min(p, L - 1) * step, c1 = min(p + 1, L - 1) * step, c2 = min(p + 2, L - 1) * step;
            // all eight operand cells first, then the six products; cells past the end of the line are masked
            const float a0 = pa[c0], b00 = pb[c0], b01 = pb[c1], b02 = pb[c2];
            const float a1 = pa[org1 + c0], b10 = pb[org1 + c0], b11 = pb[org1 + c1], b12 = pb[org1 + c2];
            const bool in0 = p < L, in1 = p + 1 < L, in2 = p + 2 < L;
            const float a0m = in0 ? a0 : 0.f, a1m = in0 ? a1 : 0.f;
            vs[v0] += a0m;
            vs[v0 + 1] += a1m;
            acc[m0 + 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0m, in0 ? b00 : 0.f, acc[m0 + 0], 0, 0, 0);
            acc[m0 + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0m, in1 ? b01 : 0.f, acc[m0 + 1], 0, 0, 0);
            acc[m0 + 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0m, in2 ? b02 : 0.f, acc[m0 + 2], 0, 0, 0);
            acc[m0 + 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1m, in0 ? b10 : 0.f, acc[m0 + 3], 0, 0, 0);
            acc[m0 + 4] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1m, in1 ? b11 : 0.f, acc[m0 + 4], 0, 0, 0);
            acc[m0 + 5] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1m, in2 ? b12 : 0.f, acc[m0 + 5], 0, 0, 0);
        }
    };

#pragma unroll
    for (int j = 0; j < DEPTH; ++j)
        if (n0 + j < n1) fetch(j, n0 + j);
    for (int nb = n0; nb < n1; nb += DEPTH) {
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            const int n = nb + j;
            if (n >= n1) break;
            __syncthreads();                          // the products on the previous image are done
#pragma unroll
            for (int k = 0; k < NT; ++k)
                if (gofs[k] >= 0) *reinterpret_cast<floatx4 *>(img + lofs[k]) = regs[j][k];
            __syncthreads();
            if (n + DEPTH < n1) fetch(j, n + DEPTH);  // refill this register set: in flight for DEPTH images
            float av[4], bv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int cell = ((q & 2) ? (H - 1) * W : 0) + ((q & 1) ? W - 1 : 0);
                av[q] = pa[cell];
                bv[q] = pb[cell];
            }
            lines(W, 1, (H - 1) * W, 0, 0);           // rows 0 and H-1: k runs along the row
            lines(H, W, W - 1, 6, 2);                 // columns 0 and W-1: k runs down the column
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // a corner is a single cell: only k = 0 of the step carries it
                const float a = kk == 0 ? av[q] : 0.f;
                vs[4 + q] += a;
                acc[12 + q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv[q], acc[12 + q], 0, 0, 0);
            }
        }
    }

#pragma unroll
    for (int m = 0; m < C3_BQ; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) Bm[((long)m * C + 16 * ct + 4 * kk + v) * C + 16 * ctp + lr] = acc[m][v];
#pragma unroll
    for (int m = 0; m < C3_BV; ++m) {
        float sm = vs[m];
        sm += __shfl_xor(sm, 16);
        sm += __shfl_xor(sm, 32);
        if (ctp == 0 && kk == 0) Bv[m * C + 16 * ct + lr] = sm;
    }
}

// Sums over the parts (lag matrices, channel sums) and over the image chunks (border terms), fixed order.  A thread takes four
// consecutive elements of a matrix.  A network of few layers has many parts a layer (256 of one layer of 16 channels, whose 13
// matrices are 832 threads' work): from 32 parts on, 16 threads share an element (346 -> 72 us for
// the factor of one layer of 16 x 32 x 32, batch 128, together with the sum over the wavefronts of a block; the 108 layers of
// a network of three widths, 3 to 7 parts each, take 21 us without).
constexpr int C3_SLICES = 16;
constexpr int corr3_slices(int parts) { return parts >= 32 ? C3_SLICES : 1; }
inline int corr3_sum_blocks(int C, int parts, int &fblocks)
{
    fblocks = (C3_LAGS * C * C / 4 * corr3_slices(parts) + 255) / 256;
    return fblocks + (C3_BQ * C * C / 4 + (1 + C3_BV) * C + 255) / 256;
}

__global__ __launch_bounds__(256) void corr3_sum_kernel(const CorrTable tab)
{
    __shared__ floatx4 slice_sum[C3_SLICES][256 / C3_SLICES];
    const CorrProb &pr = tab.p[corr_locate(tab, blockIdx.x)];
    const int C = pr.C, cc = C * C;
    const long nF = (long)C3_LAGS * cc, nB = (long)C3_BQ * cc;
    const long qF = nF / 4, qB = nB / 4;            // matrices: four consecutive elements (one row) per thread
    const int local = blockIdx.x - pr.blk_start;
    auto store_both = [&](float *dst, float *dstT, long e, const floatx4 &v) {
        *reinterpret_cast<floatx4 *>(dst + e) = v;
        const int l = (int)(e / cc), rem = (int)(e - (long)l * cc), c = rem / C, c2 = rem - c * C;
        float *t = dstT + (long)l * cc + (long)c2 * C + c;
#pragma unroll
        for (int i = 0; i < 4; ++i) t[(long)i * C] = v[i];
    };
    if (local < pr.fblocks) {
        const int sl = corr3_slices(pr.parts);
        const int first = sl == 1 ? 0 : threadIdx.x / (256 / C3_SLICES);
        const long q = sl == 1 ? (long)local * 256 + threadIdx.x : (long)local * (256 / C3_SLICES) + threadIdx.x % (256 / C3_SLICES);
        const long e = 4 * min(q, qF - 1);
        // the matrix of lag 0 is symmetric up to the order of its piece products: both halves from the lower one
        const int row = (int)(e / C), col = (int)(e - (long)row * C);
        const bool mirrored = e < cc && col + 3 > row;
        auto part = [&](int p) -> floatx4 {
            const float *src = pr.Fp + (long)p * nF;
            if (!mirrored) return *reinterpret_cast<const floatx4 *>(src + e);
            floatx4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = src[(long)max(row, col + i) * C + min(row, col + i)];
            return v;
        };
        // four interleaved running sums (fixed order) keep loads in flight
        floatx4 a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        int p = first;
        for (; p + 3 * sl < pr.parts; p += 4 * sl)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] += part(p + j * sl);
        for (; p < pr.parts; p += sl) a[0] += part(p);
        floatx4 sum = (a[0] + a[1]) + (a[2] + a[3]);
        if (sl > 1) {
            slice_sum[first][threadIdx.x % (256 / C3_SLICES)] = sum;
            __syncthreads();
            if (first > 0) return;
            for (int k = 1; k < C3_SLICES; ++k) sum += slice_sum[k][threadIdx.x];
        }
        if (q < qF) store_both(pr.Fs, pr.FsT, e, sum);
        return;
    }
    const long q = (long)(local - pr.fblocks) * 256 + threadIdx.x;
    if (q < qB) {
        const long i = 4 * q;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < C3_CHUNKS; ++k) sum += *reinterpret_cast<const floatx4 *>(pr.Bp + (long)k * nB + i);
        store_both(pr.Bs, pr.BsT, i, sum);
    } else if (q < qB + C) {
        const long c = q - qB;
        float sum = 0.f;
#pragma unroll 8
        for (int p = 0; p < pr.parts; ++p) sum += pr.Fp[(long)pr.parts * nF + (long)p * C + c];
        pr.Fs[nF + c] = sum;
    } else if (q < qB + C + C3_BV * C) {
        const long i = q - qB - C;
        float sum = 0.f;
        for (int k = 0; k < C3_CHUNKS; ++k) sum += pr.Bp[(long)C3_CHUNKS * nB + (long)k * (C3_BV * C) + i];
        pr.Bs[nB + i] = sum;
    }
}

// Assembly of A from the lag matrices and the border terms, with scale and running average.  A wavefront
// takes three rows of A (input channel c, kernel row i) and 64 partner channels, lane c2 the entries of the pair (c, c2):
// every lag matrix and border matrix is read once at [c][c2] and once at [c2][c] (F(-d)[c][c'] = F(d)[c'][c]; the
// summation kernel leaves a transposed copy, so both reads run along rows),
// and which of them enters element ((i,j), (i',j')) is known at compile time.  The nine values of a lane per
// row go to an LDS strip and are read back along the row of A, so the old factor is read and the new one
// stored in whole rows; both triangles are computed, nothing is stored transposed.  The wavefront after the
// last channel writes the bias row.
constexpr int C3_ARW = 4;          // row triples (wavefronts) per workgroup

template <int I>
__device__ __forceinline__ void corr3_assemble_rows(const CorrProb &pr, int c, int cb, int lane, float *st)
{
    const int C = pr.C, d = 9 * C, dF = d + pr.has_bias;
    const int x0 = 9 * 64 * cb, xn = min(9 * 64, d - x0);             // columns of this block of partner channels
    const float *Fs = pr.Fs, *Ts = pr.Fs + (long)C3_LAGS * C * C;
    const float *Bs = pr.Bs, *Bv = pr.Bs + (long)C3_BQ * C * C;
    const float wnew = (1.0f - pr.decay) * pr.scale, decay = pr.decay;
    const int c2 = 64 * cb + lane < C ? 64 * cb + lane : 0;          // idle lanes repeat a valid address
    // the old rows (clamped addresses: no branch, all loads in flight at once) and the bias column entries:
    // column sum of patch column (c, I, j) = all pixels minus the removed row / column plus the corner
    float old[3][9], oldb[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const float *row = pr.F + (long)(9 * c + 3 * I + j) * dF;
#pragma unroll
        for (int k = 0; k < 9; ++k) old[j][k] = row[min(x0 + lane + 64 * k, dF - 1)];
        float t = Ts[c];
        if (I != 1) t -= Bv[(I == 0 ? 1 : 0) * C + c];
        if (j != 1) t -= Bv[(j == 0 ? 3 : 2) * C + c];
        if (I != 1 && j != 1) t += Bv[(4 + (I == 0 ? 2 : 0) + (j == 0 ? 1 : 0)) * C + c];
        oldb[j] = decay * row[dF - 1] + wnew * t;
    }
    float Fp[C3_LAGS], Fn[C3_LAGS], Rp[4][3], Rn[4][3], Cq[4];
#pragma unroll
    for (int l = 0; l < C3_LAGS; ++l) {
        Fp[l] = Fs[((long)l * C + c) * C + c2];
        Fn[l] = pr.FsT[((long)l * C + c) * C + c2];
    }
#pragma unroll
    for (int sd = 0; sd < 4; ++sd)
#pragma unroll
        for (int lag = 0; lag < 3; ++lag) {
            Rp[sd][lag] = Bs[((long)(3 * sd + lag) * C + c) * C + c2];
            Rn[sd][lag] = pr.BsT[((long)(3 * sd + lag) * C + c) * C + c2];
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) Cq[q] = Bs[((long)(12 + q) * C + c) * C + c2];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int ij2 = 0; ij2 < 9; ++ij2) {
            const int i2 = ij2 / 3, j2 = ij2 - 3 * i2;
            const int di = i2 - I, dj = j2 - j;
            const bool pos = di > 0 || (di == 0 && dj >= 0);
            const int adi = pos ? di : -di, adj = pos ? dj : -dj;
            const int l = adi == 0 ? adj : (adi == 1 ? 5 + adj : 10 + adj);
            float val = pos ? Fp[l] : Fn[l];
            if (i2 == I && I != 1) {          // removed row a* = H-1 (i = 0) or 0 (i = 2); lag j2 - j along the row
                const int sd = I == 0 ? 1 : 0;
                val -= dj >= 0 ? Rp[sd][dj >= 0 ? dj : 0] : Rn[sd][dj < 0 ? -dj : 0];
            }
            if (j2 == j && j != 1) {
                const int sd = j == 0 ? 3 : 2;
                val -= di >= 0 ? Rp[sd][di >= 0 ? di : 0] : Rn[sd][di < 0 ? -di : 0];
            }
            if (i2 == I && I != 1 && j2 == j && j != 1) val += Cq[(I == 0 ? 2 : 0) + (j == 0 ? 1 : 0)];
            st[9 * lane + ij2] = val;
        }
        __builtin_amdgcn_wave_barrier();       // LDS serves a wavefront's accesses in order: the reads below see the row
        float *row = pr.F + (long)(9 * c + 3 * I + j) * dF;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if (lane + 64 * k < xn) row[x0 + lane + 64 * k] = decay * old[j][k] + wnew * st[lane + 64 * k];
        if (pr.has_bias && lane == 0 && cb == 0) row[d] = oldb[j];
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ __launch_bounds__(256) void corr3_assemble_kernel(const CorrTable tab)
{
    __shared__ float strip[C3_ARW][9 * 64 + 4];
    const CorrProb &pr = tab.p[corr_locate(tab, blockIdx.x)];
    const int C = pr.C, d = 9 * C, dF = d + pr.has_bias;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // row triple and block of 64 partner channels: the same for the whole wavefront
    const int cbs = (C + 63) / 64, unit = C3_ARW * (blockIdx.x - pr.blk_start) + w, rt = unit / cbs, cb = unit - rt * cbs;
    const int c = rt / 3, i = rt - 3 * c;
    if (c > C || (c == C && (i > 0 || cb > 0 || !pr.has_bias))) return;
    if (c == C) {
        const float *Ts = pr.Fs + (long)C3_LAGS * C * C, *Bv = pr.Bs + (long)C3_BQ * C * C;
        const float wnew = (1.0f - pr.decay) * pr.scale;
        float *row = pr.F + (long)d * dF;
        for (int x = lane; x < dF; x += 64) {
            float val;
            if (x == d) {
                val = (float)((long)pr.B * pr.H * pr.W);
            } else {
                const int cc = x / 9, ij = x - 9 * cc, ii = ij / 3, jj = ij - 3 * ii;
                val = Ts[cc];
                if (ii != 1) val -= Bv[(ii == 0 ? 1 : 0) * C + cc];
                if (jj != 1) val -= Bv[(jj == 0 ? 3 : 2) * C + cc];
                if (ii != 1 && jj != 1) val += Bv[(4 + (ii == 0 ? 2 : 0) + (jj == 0 ? 1 : 0)) * C + cc];
            }
            row[x] = pr.decay * row[x] + wnew * val;
        }
        return;
    }
    if (i == 0) corr3_assemble_rows<0>(pr, c, cb, lane, strip[w]);
    else if (i == 1) corr3_assemble_rows<1>(pr, c, cb, lane, strip[w]);
    else corr3_assemble_rows<2>(pr, c, cb, lane, strip[w]);
}

}  // namespace kfac
