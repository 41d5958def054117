// fp32 MFMA GEMM of the form  C = A^T B  (both operands stored K-major), used
// for the two-sided preconditioning  P = G_inv * grad * A_inv  (Eq. 5 / rhs of
// Eq. 12 of the DP-KFAC paper): U^T = grad^T G_inv, then P = (U^T)^T A_inv, both
// with row-major outputs, no operand is ever read with a strided K; and for the
// panel products and rank-k updates of the blocked inversion.  Wide products
// go to the wave-unit kernel (gemm_wave.hpp), the rest to the two block-tile kernels
// below.
#include <type_traits>
#include "gemm_wave.hpp"
#include "gemm_split.hpp"

#include <algorithm>
#include <vector>

namespace kfac {

struct GemmProb {
    const float *A;
    const float *B;
    float *C;
    long lda, ldb, ldc;
    int M, N, K;
    int tm, tn;       // tiles per side
    int blk_start;
    int mode;
    int p0, p1;
    long doff;
    int vecA, vecB;
    const float *rv, *cv;   // kStoreDiv
    float gamma;
    const int *gate;        // null, or two float bit patterns: leave C alone unless their product exceeds gate_cond
    float gate_cond;
    const float *D;         // kSubFrom
    long ldd;
};

// A launch covers up to kMaxGemmProblems products (a 14 KB kernel argument): the preconditioning of a whole
// network is then two launches, and the k-loop latency of a small product is paid once, not once per group of
// layers.  The first block of every product sits in a compact array of its own, searched by bisection.
constexpr int kMaxGemmProblems = 128;

struct GemmTable {
    int count;
    int starts[kMaxGemmProblems];
    GemmProb p[kMaxGemmProblems];
};

template <class T>
__global__ __launch_bounds__(T::NT) void gemm_tn_kernel(const GemmTable tab)
{
    __shared__ float lds[2][2][T::PANEL];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / T::NW, wn = wave % T::NW;

    int pi = 0, hi = tab.count - 1;
    while (pi < hi) {
        const int mid = (pi + hi + 1) >> 1;
        if ((int)blockIdx.x >= tab.starts[mid]) pi = mid;
        else hi = mid - 1;
    }
    const GemmProb &pr = tab.p[pi];
    if (pr.gate && !(__int_as_float(pr.gate[0]) * __int_as_float(pr.gate[1]) > pr.gate_cond)) return;   // uniform
    const int local = blockIdx.x - pr.blk_start;
    int bi, bj;
    if (pr.mode == kSubLowerSkip) {
        tri_decode(local, bi, bj);
    } else {
        bi = local / pr.tn;
        bj = local - bi * pr.tn;
    }
    const int m0 = bi * T::BM, n0 = bj * T::BM;

    Operand opA, opB;
    opA.x = pr.A; opA.K = pr.K; opA.ld = pr.lda; opA.d = pr.M; opA.hw = 1; opA.ctot = 0; opA.vec = pr.vecA;
    opB.x = pr.B; opB.K = pr.K; opB.ld = pr.ldb; opB.d = pr.N; opB.hw = 1; opB.ctot = 0; opB.vec = pr.vecB;

    floatx4 acc[T::WT][T::WT];
#pragma unroll
    for (int i = 0; i < T::WT; ++i)
#pragma unroll
        for (int j = 0; j < T::WT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // The panels are fetched D stages ahead into a ring of register sets, so that a stage waits for loads
    // issued D stages earlier: the short, latency-bound products (a few workgroups per matrix, each walking
    // the whole depth) live on that.  Set r holds stage t with t mod D = r; it is free again once that stage
    // has been written to LDS.  The large tiles keep one set (registers).
    constexpr int D = T::BM <= 32 ? 3 : 1;
    const long ktiles = (pr.K + T::KT - 1) / T::KT;
    auto k_loop = [&](auto vec_a, auto vec_b) {
        constexpr bool VA = decltype(vec_a)::value, VB = decltype(vec_b)::value;
        floatx4 sa[D][T::PASSES], sb[D][T::PASSES];
#pragma unroll
        for (int r = 0; r < D; ++r) {       // stages past the depth re-read the last rows and are never written to LDS
            fetch_rows_clamped<T, 0, VA>(sa[r], opA, (long)r * T::KT, m0, tid);
            fetch_rows_clamped<T, 0, VB>(sb[r], opB, (long)r * T::KT, n0, tid);
            __builtin_amdgcn_sched_barrier(0);      // issued in the order the loop consumes them
        }
        commit_rows_masked<T>(sa[0], opA, 0, m0, lds[0][0], tid);
        commit_rows_masked<T>(sb[0], opB, 0, n0, lds[0][1], tid);
        __syncthreads();
        for (long t0 = 0; t0 < ktiles; t0 += D) {
#pragma unroll
            for (int r = 0; r < D; ++r) {
                const long t = t0 + r;
                if (t >= ktiles) break;
                const int cur = (int)(t & 1);
                fetch_rows_clamped<T, 0, VA>(sa[r], opA, (t + D) * T::KT, m0, tid);
                fetch_rows_clamped<T, 0, VB>(sb[r], opB, (t + D) * T::KT, n0, tid);
                mma_stage<T, kRows, kRows, false>(lds[cur][0], lds[cur][1], wm, wn, lane, acc);
                if (t + 1 < ktiles) {
                    commit_rows_masked<T>(sa[(r + 1) % D], opA, (t + 1) * T::KT, m0, lds[cur ^ 1][0], tid);
                    commit_rows_masked<T>(sb[(r + 1) % D], opB, (t + 1) * T::KT, n0, lds[cur ^ 1][1], tid);
                }
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (opA.vec) {
        if (opB.vec) k_loop(std::true_type{}, std::true_type{});
        else k_loop(std::true_type{}, std::false_type{});
    } else {
        if (opB.vec) k_loop(std::false_type{}, std::true_type{});
        else k_loop(std::false_type{}, std::false_type{});
    }

    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
        for (int tj = 0; tj < T::WT; ++tj) {
            const int n = n0 + (wn * T::WT + tj) * 16 + lr;
            if (n >= pr.N) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + (wm * T::WT + ti) * 16 + 4 * lk + v;
                if (m >= pr.M) continue;
                const float val = acc[ti][tj][v];
                if (pr.mode == kStore) {
                    pr.C[(long)m * pr.ldc + n] = val;
                } else if (pr.mode == kStoreDiv) {
                    pr.C[(long)m * pr.ldc + n] = val / (pr.rv[m] * pr.cv[n] + pr.gamma);
                } else if (pr.mode == kSubFrom) {
                    pr.C[(long)m * pr.ldc + n] = pr.D[(long)m * pr.ldd + n] - val;
                } else if (pr.mode == kSubRect || pr.mode == kAddRect) {
                    const bool skip = ((long)n > (long)m + pr.doff) || (n >= pr.p0 && n < pr.p1);
                    if (!skip) pr.C[(long)m * pr.ldc + n] += pr.mode == kAddRect ? val : -val;
                } else {
                    const bool skip = (n > m) || (m >= pr.p0 && m < pr.p1) || (n >= pr.p0 && n < pr.p1);
                    if (!skip) pr.C[(long)m * pr.ldc + n] -= val;
                }
            }
        }
}

// Products of the blocked inversion's chain: 32 x 32 tiles, a wavefront each, on the split arithmetic (split_common.hpp) in
// the order of gemm_split_kernel: the same bits as the panel and bulk products leave, so that the next pivot block is updated
// with the very W that the rest of its matrix sees.  (With W from the fp32 MFMA, as accurate by itself, the inverse of a
// post-ReLU factor came out up to 6 % further from float64, condition number 1e4 to 1e5: the two roundings, eps |V| |P|
// each, no longer cancel.)  Operands go straight from memory to the wavefront that cuts them, four stages of 16 rows in
// flight; no LDS, no barrier.  K is a multiple of 64.  A launch of five products 256 x 256 x 256: 14 us.
__global__ __launch_bounds__(64) void gemm_chain_kernel(const GemmTable tab)
{
    int pi = 0, hi = tab.count - 1;
    while (pi < hi) {
        const int mid = (pi + hi + 1) >> 1;
        if ((int)blockIdx.x >= tab.starts[mid]) pi = mid;
        else hi = mid - 1;
    }
    const GemmProb &pr = tab.p[pi];
    if (pr.gate && !(__int_as_float(pr.gate[0]) * __int_as_float(pr.gate[1]) > pr.gate_cond)) return;
    const int local = blockIdx.x - pr.blk_start, bi = local / pr.tn;
    const int m0 = 32 * bi, n0 = 32 * (local - bi * pr.tn), M = pr.M, N = pr.N, nst = pr.K / 16;
    const bool lower = pr.mode == kSubRect || pr.mode == kAddRect;
    if (lower && (long)n0 > (long)min(m0 + 31, M - 1) + pr.doff) return;       // wholly above the line n = m + doff
    const int lane = threadIdx.x, lr = lane & 31, lg = lane >> 5;
    const unsigned pa = (unsigned)pr.lda * 4u, pb = (unsigned)pr.ldb * 4u;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.A), 0, (int)((long)pr.K * pr.lda * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.B), 0, (int)((long)pr.K * pr.ldb * 4), 0x00020000);
    // columns past the edge repeat the last one: their results are not stored
    const unsigned ca = (unsigned)min(m0 + lr, M - 1) * 4u, cb = (unsigned)min(n0 + lr, N - 1) * 4u;
    const unsigned ao = ca + 8u * (unsigned)lg * pa, bo = cb + 8u * (unsigned)lg * pb;
    float a[4][8], b[4][8];                   // rows 16 g + 8 lg + e
    auto load = [&](int set, int g) {
        const int gg = min(g, nst - 1);       // past the end: the last stage again, not used
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a[set][e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, ao, (unsigned)(16 * gg + e) * pa, 0));
            b[set][e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, bo, (unsigned)(16 * gg + e) * pb, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pieces = [&](sbf16x8 (&f)[3], const float (&x)[8]) {
        float x0[4] = {x[0], x[1], x[2], x[3]}, x1[4] = {x[4], x[5], x[6], x[7]};
        SplitCut k0, k1;
        k0.scale(x0); k1.scale(x1);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            k0.half(x0, 0, 4); k1.half(x1, 0, 4);
            const suint2 u = k0.pack(), v = k1.pack();
            f[p] = __builtin_bit_cast(sbf16x8, suint4{u.x, u.y, v.x, v.y});
            k0.top(0, 4); k1.top(0, 4);
            k0.rest(x0, 0, 4); k1.rest(x1, 0, 4);
        }
        const suint2 u = k0.pack_last(x0), v = k1.pack_last(x1);
        f[2] = __builtin_bit_cast(sbf16x8, suint4{u.x, u.y, v.x, v.y});
    };
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) load(t, t);
    sbf16x8 A[2][3], B[2][3];
    pieces(A[0], a[0]);
    pieces(B[0], b[0]);
    load(0, 4);
    for (int g = 0; g < nst; g += 4)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // the cut of the next stage between the products of this one, which wait for each other
            pieces(A[(t + 1) & 1], a[(t + 1) & 3]);
            pieces(B[(t + 1) & 1], b[(t + 1) & 3]);
            constexpr int pieceA[6] = {2, 1, 1, 0, 0, 0}, pieceB[6] = {0, 1, 0, 2, 1, 0};
#pragma unroll
            for (int q = 0; q < 6; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t & 1][pieceA[q]], B[t & 1][pieceB[q]], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 23, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            load((t + 1) & 3, g + t + 5);
        }
    float unscale = kSplitUnscale, t = 0.f;   // t stays 0 unless something is infinite or NaN
#pragma unroll
    for (int v = 0; v < 16; ++v) t = __builtin_fmaf(acc[v], 0.f, t);
    if (__any(t != 0.f)) {                    // what fp32 arithmetic gives
        unscale = 1.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        for (int k = 0; k < 16 * nst; k += 2) {
            const float x = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, ca + (unsigned)(k + lg) * pa, 0, 0));
            const float y = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, cb + (unsigned)(k + lg) * pb, 0, 0));
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
        }
    }
    const int n = n0 + lr;
    const float *from = pr.mode == kSubFrom ? pr.D : pr.C;
    const long ldf = pr.mode == kSubFrom ? pr.ldd : pr.ldc;
    const float sign = pr.mode == kStore || pr.mode == kAddRect ? unscale : -unscale;
    float old[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + 8 * (v >> 2) + 4 * lg + (v & 3);
        old[v] = pr.mode != kStore && m < M && n < N ? from[(long)m * ldf + n] : 0.f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + 8 * (v >> 2) + 4 * lg + (v & 3);
        if (m < M && n < N && (!lower || (long)n <= (long)m + pr.doff)) pr.C[(long)m * pr.ldc + n] = __builtin_fmaf(sign, acc[v], old[v]);
    }
}

// 64 x 64 tiles of the same products for the launches that are bound by the latency of one tile: a few workgroups per
// matrix, each walking the whole depth (small preconditioning products).  The four wavefronts split K (chunks of 16 in turn), every one computes the whole tile: a lane loads 16 bytes
// of a row of either operand, which are one column each of four interleaved MFMA tiles, straight into the registers the
// MFMA reads, two chunks ahead; no LDS and no barrier until the four parts are added in wavefront order.  At K = 256 a
// tile takes 9 us where the staged form with all wavefronts on one K stage (16 stages, an LDS round trip and a barrier
// each) took 21; the pieces of an operand past its edge feed outputs that are not stored.
typedef float gmfloat4 __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256, 2) void gemm_direct_kernel(const GemmTable tab)
{
    __shared__ floatx4 lds[4 * 3 * 4 * 64];
    int pi = 0, hi = tab.count - 1;
    while (pi < hi) {
        const int mid = (pi + hi + 1) >> 1;
        if ((int)blockIdx.x >= tab.starts[mid]) pi = mid;
        else hi = mid - 1;
    }
    const GemmProb &pr = tab.p[pi];
    if (pr.gate && !(__int_as_float(pr.gate[0]) * __int_as_float(pr.gate[1]) > pr.gate_cond)) return;   // uniform
    const int local = blockIdx.x - pr.blk_start;
    int bi, bj;
    if (pr.mode == kSubLowerSkip) {
        tri_decode(local, bi, bj);
    } else {
        bi = local / pr.tn;
        bj = local - bi * pr.tn;
    }
    const int m0 = bi * 64, n0 = bj * 64, M = pr.M, N = pr.N, K = pr.K;
    const bool lower = pr.mode == kSubLowerSkip || pr.mode == kSubRect || pr.mode == kAddRect;
    if (lower && (long)n0 > (long)min(m0 + 63, M - 1) + pr.doff) return;      // wholly above the line n = m + doff
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    typedef int gint4 __attribute__((ext_vector_type(4)));
    // the host checked: below 2 GiB; rows past K are past the end and read as zero
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.A), 0, (int)((long)K * pr.lda * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.B), 0, (int)((long)K * pr.ldb * 4), 0x00020000);
    const unsigned pa = (unsigned)pr.lda * 4u, pb = (unsigned)pr.ldb * 4u;
    // a lane whose four columns all lie past the edge reads the tile's first ones
    const unsigned ao = (unsigned)(m0 + (m0 + 4 * lr < M ? 4 * lr : 0)) * 4u, bo = (unsigned)(n0 + (n0 + 4 * lr < N ? 4 * lr : 0)) * 4u;
    floatx4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](gint4 (&a)[4], gint4 (&b)[4], int k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int kk = k + 4 * e + lk;
            const unsigned ro = kk < K ? (unsigned)kk * pa + ao : 0x80000000u, so = kk < K ? (unsigned)kk * pb + bo : 0x80000000u;
            a[e] = __builtin_bit_cast(gint4, __builtin_amdgcn_raw_buffer_load_b128(ra, ro, 0, 0));
            b[e] = __builtin_bit_cast(gint4, __builtin_amdgcn_raw_buffer_load_b128(rb, so, 0, 0));
        }
    };
    auto multiply = [&](const gint4 (&a)[4], const gint4 (&b)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(a[e][i]), __int_as_float(b[e][t]), acc[i][t], 0, 0, 0);
    };
    gint4 a0[4], b0[4], a1[4], b1[4];
    load(a0, b0, 16 * w);
    __builtin_amdgcn_sched_barrier(0);
    load(a1, b1, 16 * w + 64);
    __builtin_amdgcn_sched_barrier(0);
    for (int k = 16 * w; k < K; k += 128) {
        multiply(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        load(a0, b0, k + 128);
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        load(a1, b1, k + 192);
        __builtin_amdgcn_sched_barrier(0);
    }
    // the parts: wavefront t sums MFMA column tile t
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t != w) {
            floatx4 *d = lds + ((t * 3 + (w < t ? w : w - 1)) * 4) * 64 + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i * 64] = acc[i][t];
        }
    __syncthreads();
    floatx4 sum[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        floatx4 own = acc[i][0];
#pragma unroll
        for (int t = 1; t < 4; ++t)
            if (t == w) own = acc[i][t];
        sum[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) sum[i] += ww == w ? own : lds[((w * 3 + (ww < w ? ww : ww - 1)) * 4 + i) * 64 + lane];
    }
    __syncthreads();
    constexpr int PO = 68;
    float *o = reinterpret_cast<float *>(lds);          // the tile: row 4 (4 lk + v) + i, column 4 lr + w
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[(4 * (4 * lk + v) + i) * PO + 4 * lr + w] = sum[i][v];
    __syncthreads();
    // 16 lanes along a row, four columns each: all old values before the first store
    const int mr = tid >> 4, c = 4 * (tid & 15), n = n0 + c;
    floatx4 old[4];
    const bool reads = lower || pr.mode == kSubFrom;
    const float *from = pr.mode == kSubFrom ? pr.D : pr.C;
    const long ldf = pr.mode == kSubFrom ? pr.ldd : pr.ldc;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + mr + 16 * r;
        old[r] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (reads && m < M && n < N) {
            const float *src = from + (long)m * ldf + n;
            if (n + 3 < N) old[r] = *reinterpret_cast<const gmfloat4 *>(src);
            else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (n + e < N) old[r][e] = src[e];
            }
        }
    }
    const bool rows_skip = pr.mode == kSubLowerSkip;
    const float sign = pr.mode == kStore || pr.mode == kStoreDiv || pr.mode == kAddRect ? 1.f : -1.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + mr + 16 * r;
        if (m >= M || (rows_skip && m >= pr.p0 && m < pr.p1)) continue;
        floatx4 val = *reinterpret_cast<const floatx4 *>(o + (mr + 16 * r) * PO + c);
        if (pr.mode == kStoreDiv) {
            const float rv = pr.rv[m];
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = val[e] / (rv * pr.cv[min(n + e, N - 1)] + pr.gamma);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e] = __builtin_fmaf(sign, val[e], old[r][e]);
        const long last = lower ? min((long)N - 1, (long)m + pr.doff) : N - 1;
        float *dst = pr.C + (long)m * pr.ldc + n;
        const bool band = lower && n + 3 >= pr.p0 && n < pr.p1;       // columns of the pivot band are left alone
        if (n + 3 <= last && !band) *reinterpret_cast<gmfloat4 *>(dst) = val;
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e <= last && !(lower && n + e >= pr.p0 && n + e < pr.p1)) dst[e] = val[e];
        }
    }
}

namespace {

const int kBms[] = {128, 144, 64, 32};

int choose_bm(int M, int N, bool square_lower)
{
    const long force = square_lower ? tuning().update_bm : tuning().gemm_bm;
    if (force)
        for (int i = 0; i < 4; ++i)
            if (kBms[i] == force) return i;
    int best = 0;
    double best_cost = 1e300;
    for (int i = 0; i < 4; ++i) {
        const long bm = kBms[i];
        const long tm = (M + bm - 1) / bm, tn = (N + bm - 1) / bm;
        const double tiles = square_lower ? (double)tm * (tm + 1) / 2 : (double)tm * tn;
        const double penalty = bm >= 128 ? 1.0 : (bm >= 64 ? 1.15 : 1.4);
        const double cost = tiles * bm * bm * penalty;
        if (cost < best_cost - 1e-9) { best_cost = cost; best = i; }
    }
    return best;
}

hipError_t launch_done(const GemmTable &tab)
{
    double flops = 0.0;
    for (int k = 0; k < tab.count; ++k) {
        const GemmProb &p = tab.p[k];
        if (p.gate) continue;       // may be skipped on the device: not counted
        if (p.mode != kSubLowerSkip) { flops += 2.0 * p.M * p.N * p.K; continue; }
        const double live = (double)p.M - (double)(std::min(p.p1, p.M) - p.p0);
        flops += live * (live + 1.0) * p.K;
    }
    timing_work(flops, flops);
    return hipGetLastError();
}

template <class T>
hipError_t launch_one(const GemmTable &tab, int blocks, hipStream_t s)
{
    KFAC_LAUNCH(KFAC_K_GEMM, s, (gemm_tn_kernel<T>), dim3(blocks), dim3(T::NT), 0, tab);
    return launch_done(tab);
}

hipError_t launch_direct(const GemmTable &tab, int blocks, hipStream_t s)
{
    KFAC_LAUNCH(KFAC_K_GEMM, s, gemm_direct_kernel, dim3(blocks), dim3(256), 0, tab);
    return launch_done(tab);
}

// the products of the blocked inversion's chain: K a multiple of 64, operands below 2 GiB (pivot blocks of 64 to 512 rows).
// (Never in a timed pass, which keeps everything on one stream: no chain.  Hence the class of the other small products.)
hipError_t chain_launch(const GemmJob *jobs, int n, hipStream_t s)
{
    for (int i0 = 0; i0 < n; i0 += kMaxGemmProblems) {
        GemmTable tab;
        tab.count = std::min(kMaxGemmProblems, n - i0);
        int blocks = 0;
        for (int k = 0; k < tab.count; ++k) {
            const GemmJob &j = jobs[i0 + k];
            GemmProb &p = tab.p[k];
            p = GemmProb{};
            p.A = j.A; p.B = j.B; p.C = j.C;
            p.lda = j.lda; p.ldb = j.ldb; p.ldc = j.ldc;
            p.M = j.M; p.N = j.N; p.K = j.K;
            p.tm = (j.M + 31) / 32;
            p.tn = (j.N + 31) / 32;
            p.mode = j.mode; p.doff = j.doff;
            p.gate = j.gate; p.gate_cond = j.gate_cond;
            p.D = j.D; p.ldd = j.ldd;
            p.blk_start = tab.starts[k] = blocks;
            blocks += p.tm * p.tn;
        }
        KFAC_LAUNCH(KFAC_K_GEMM, s, gemm_chain_kernel, dim3(blocks), dim3(64), 0, tab);
        hipError_t e = launch_done(tab);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

namespace {
// flops of the definition of a product (the lower-triangle update counts the entries it touches)
double gemm_job_flops(const GemmJob &j)
{
    if (j.mode == kSubRect || j.mode == kAddRect) {
        // rows m = 0..M-1 touch the columns n <= min(N - 1, m + doff) outside [p0, p1)
        double cnt = 0.0;
        for (int m = 0; m < j.M; ++m) {
            const long hi = std::min<long>(j.N - 1, m + j.doff);
            if (hi < 0) continue;
            long c = hi + 1;
            const long a = std::max<long>(0, j.p0), b = std::min<long>(hi + 1, j.p1);
            if (b > a) c -= b - a;
            cnt += (double)c;
        }
        return 2.0 * cnt * j.K;
    }
    if (j.mode != kSubLowerSkip) return 2.0 * j.M * j.N * j.K;
    const double live = (double)j.M - (double)(std::min(j.p1, j.M) - j.p0);
    return live * (live + 1.0) * j.K;
}

// Products wide enough to fill 144-wide macro tiles go to the wave-unit kernel.  A lower-triangular
// update qualifies only when its untouched band starts and ends on macro-tile boundaries.
bool wave_gemm_eligible(const GemmJob &j)
{
    if (!tuning().use_wave_gemm || j.mode == kStoreDiv || j.mode == kSubRect || j.mode == kAddRect ||
        j.mode == kSubFrom || j.gate)
        return false;
    if (j.M < 100 || j.N < 100 || j.K < 16) return false;
    if ((long)j.K * j.lda * 4 > 0x7fffffffl || (long)j.K * j.ldb * 4 > 0x7fffffffl) return false;
    if (((uintptr_t)j.A) % 4 || ((uintptr_t)j.B) % 4) return false;
    if (j.mode == kSubLowerSkip)
        return j.M == j.N && j.p0 % W_MT == 0 && (j.p1 % W_MT == 0 || j.p1 >= j.M);
    return true;
}

hipError_t wave_gemm_launch(const GemmJob *jobs, const std::vector<int> &idx, hipStream_t s)
{
    GemmWTable tab;
    tab.count = 0;
    long blocks = 0;
    double wflops = 0.0;
    auto flush = [&]() -> hipError_t {
        if (tab.count == 0) return hipSuccess;
        // Contiguous tile ranges per XCD pay when a launch spans many problems of similar depth (each XCD
        // then works on a few matrices).  With mixed depths the long workgroups would pile up on one
        // XCD, and with a handful of problems the round-robin order measured as good or better.
        int kmin = tab.p[0].K, kmax = tab.p[0].K;
        for (int k = 1; k < tab.count; ++k) {
            kmin = std::min(kmin, tab.p[k].K);
            kmax = std::max(kmax, tab.p[k].K);
        }
        tab.xcd_remap = (tab.count >= tuning().gemm_xcd_remap_min && 2 * kmax <= 3 * kmin) ? 1 : 0;
        KFAC_LAUNCH(KFAC_K_GEMM_WAVE, s, gemm_wave_kernel, dim3((unsigned)blocks), dim3(256), 0, tab);
        timing_work(wflops, wflops);
        wflops = 0.0;
        tab.count = 0;
        blocks = 0;
        return hipGetLastError();
    };
    for (int i : idx) {
        const GemmJob &j = jobs[i];
        GemmWProb &p = tab.p[tab.count++];
        p.A = j.A; p.B = j.B; p.C = j.C;
        p.lda = (int)j.lda; p.ldb = (int)j.ldb; p.ldc = (int)j.ldc;
        p.M = j.M; p.N = j.N; p.K = j.K;
        p.mI = (j.M + W_MT - 1) / W_MT;
        const int nJ = (j.N + W_MT - 1) / W_MT;
        p.nJ2 = (nJ + 1) / 2;
        p.mode = j.mode; p.p0 = j.p0; p.p1 = j.p1;
        p.blk_start = (int)blocks;
        wflops += gemm_job_flops(j);
        if (j.mode == kSubLowerSkip) {
            for (int I = 0; I < p.mI; ++I) blocks += I / 2 + 1;
        } else {
            blocks += (long)p.mI * p.nJ2;
        }
        if (tab.count == kMaxProblems) {
            hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
    }
    return flush();
}
}  // namespace

namespace {
// Products that fill 256 x 128 tiles reasonably go to the split-bf16 kernel (gemm_split.hpp).
bool split_gemm_eligible(const GemmJob &j, bool wide)
{
    if (!tuning().use_split_gemm || (j.mode != kStore && j.mode != kSubLowerSkip && j.mode != kSubRect && j.mode != kAddRect))
        return false;
    const long min_m = wide && j.mode == kStore ? tuning().split_gemm_min_m : 192;
    if (j.M < min_m || j.N < 64 || j.K < 16) return false;
    // a product of a tile or two is bound by the latency of one tile's K loop and read-modify-write (55 us at
    // K = 256): the 64-wide tiles of the block-tile kernel spread it over many CUs and finish in 10-15 us
    if ((long)j.M * j.N < 4l * S_BM * S_BN) return false;
    if (j.mode == kStore && !j.wide_tiles) {
        if (j.K < (wide ? tuning().split_gemm_min_k : 1024)) return false;
        // 256 x 128 tiles: products that fill less than 40 % of them stay with the other kernels.  The split kernel does
        // a multiply-add of the definition in less than half of the fp32 MFMA's time, so that it wins with half of a
        // tile empty and with few K stages.  Preconditioning, lines M >= 192, K >= 1024, fill 60 % -> M >= 128,
        // K >= 128, 40 % (together with the K slices below): twelve 768-wide transformer blocks 3.87 -> 2.89 ms,
        // ResNet-50-shaped 1.25 -> 1.19, DenseNet-201-shaped 1.32 -> 1.15, one 700 x 500 layer 0.23 -> 0.10,
        // a 256-channel 3x3 layer 0.117 -> 0.092 ms; fill 50 %: 1.27 and 1.23 ms on the two networks.
        // The narrow lines stay for calls whose work is mostly in products too small for either: another launch
        // for one or two products of the call costs more than they gain (an update with one of seven products moved
        // 0.92 -> 0.97 ms).  So the last bits of a product can differ with what else is in its call.  Its accuracy does
        // not suffer on either route: error against float64, split / fp32 MFMA, products of a post-ReLU gradient and
        // an inverse dominated by its diagonal, 1.39e-7 / 1.44e-7 at K = 128 and 3.7e-7 / 4.1e-7 at 1023, of zero-mean
        // operands 1.6e-7 / 2.0e-7 and 4.9e-7 / 5.7e-7.
        const double tiles = (double)((j.M + S_BM - 1) / S_BM) * ((j.N + S_BN - 1) / S_BN);
        if ((double)j.M * j.N < 0.01 * (wide ? tuning().split_gemm_min_fill : 60) * tiles * S_BM * S_BN) return false;
    }
    if ((long)j.K * j.lda * 4 > 0x7fffffffl || (long)j.K * j.ldb * 4 > 0x7fffffffl) return false;
    if ((long)j.M * j.ldc * 4 > 0x7fffffffl) return false;
    if (((uintptr_t)j.A) % 4 || ((uintptr_t)j.B) % 4) return false;
    // the epilogue decides about four columns of a pivot band at a time
    if (j.mode != kStore && (j.p0 % 4 != 0 || (j.p1 % 4 != 0 && j.p1 < j.N))) return false;
    if (j.mode == kSubLowerSkip) return j.M == j.N;
    return true;
}

// whether a call takes the wide lines: with them the split kernel has at least half of the call's work.  (The K slices
// of a product count as the product does.)
bool split_gemm_wide(const GemmJob *jobs, int n)
{
    double split = 0.0, rest = 0.0;
    for (int i = 0; i < n; ++i) {
        if (!(jobs[i].M > 0 && jobs[i].N > 0 && jobs[i].K > 0)) continue;
        (split_gemm_eligible(jobs[i], true) ? split : rest) += (double)jobs[i].M * jobs[i].N * jobs[i].K;
    }
    return split >= rest;
}

hipError_t split_gemm_launch(const GemmJob *jobs, const std::vector<int> &idx, hipStream_t s, int cls = KFAC_K_GEMM_SPLIT,
                             double definition = -1.0)
{
    GemmSTable tab;
    tab.count = 0;
    long blocks = 0;
    double flops = 0.0;
    auto flush = [&]() -> hipError_t {
        if (tab.count == 0) return hipSuccess;
        // tile ranges of the XCDs, of equal cost: the K stages of a tile and about twelve more for its start and end
        double total = 0.0;
        auto cost = [&](const GemmSProb &p) { return (std::min(p.K, p.kper) + S_KT - 1) / S_KT + 12.0; };
        for (int k = 0; k < tab.count; ++k)
            total += cost(tab.p[k]) * ((k + 1 < tab.count ? tab.p[k + 1].blk_start : (int)blocks) - tab.p[k].blk_start);
        int most = 1, x = 1;
        double before = 0.0;
        tab.xcd[0] = 0;
        tab.xcd[8] = (int)blocks;
        for (int k = 0; k < tab.count; ++k) {
            const int first = tab.p[k].blk_start, n = (k + 1 < tab.count ? tab.p[k + 1].blk_start : (int)blocks) - first;
            const double c = cost(tab.p[k]);
            for (; x < 8 && total * x / 8 <= before + c * n; ++x) tab.xcd[x] = first + (int)((total * x / 8 - before) / c);
            before += c * n;
        }
        for (; x < 8; ++x) tab.xcd[x] = (int)blocks;
        for (int k = 0; k < 8; ++k) most = std::max(most, tab.xcd[k + 1] - tab.xcd[k]);
        KFAC_LAUNCH(cls, s, gemm_split_kernel, dim3((unsigned)(8 * most)), dim3(256), 0, tab);
        timing_work(definition < 0.0 ? flops : definition, 6.0 * flops);
        if (definition > 0.0) definition = 0.0;          // with the first launch
        tab.count = 0;
        blocks = 0;
        flops = 0.0;
        return hipGetLastError();
    };
    for (int i : idx) {
        const GemmJob &j = jobs[i];
        GemmSProb &p = tab.p[tab.count++];
        p.A = j.A; p.B = j.B; p.C = j.C;
        p.lda = (int)j.lda; p.ldb = (int)j.ldb; p.ldc = (int)j.ldc;
        p.M = j.M; p.N = j.N; p.K = j.K;
        p.tI = (j.M + S_BM - 1) / S_BM;
        p.tJ = (j.N + S_BN - 1) / S_BN;
        p.mode = j.mode; p.p0 = j.p0; p.p1 = j.p1;
        p.doff = (int)std::min<long>(j.doff, 1l << 30);
        if (j.mode == kSubLowerSkip) p.doff = 0;
        p.gate = j.gate; p.gate_cond = j.gate_cond;
        p.blk_start = (int)blocks;
        tab.starts[tab.count - 1] = (int)blocks;
        p.tiles = 0;
        for (int I = 0; I < p.tI; ++I) p.tiles += split_row_len(p.mode, p.tJ, p.doff, I);
        p.kper = j.kslices > 1 ? j.kper : j.K;
        p.cstride = j.cstride;
        p.abytes = (int)(j.abytes > 0 ? j.abytes : (long)j.K * j.lda * 4);
        blocks += (long)p.tiles * std::max(1, j.kslices);
        if (!j.gate) flops += gemm_job_flops(j);       // a gated product may be skipped on the device: not counted
        if (tab.count == kMaxGemmS) {
            hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
    }
    return flush();
}
}  // namespace

namespace {
// K slices of deep products.  A call with few 256 x 128 tiles, some of them hundreds of K stages deep, leaves most
// compute units with one long workgroup and nothing to pack beside it (three 512 x 4609 x 4609 products: 222 tiles
// of 289 stages on 256 units).  Such a product is cut into K slices: slice 0 stores into C, the others into
// partial matrices in the workspace, and a reduction adds them to C in slice order (a fixed order: the result
// does not depend on the schedule).  The partials are M x N, small beside the K x N operand that is read.  The slices
// of a call are as deep as leaves about 512 workgroups of equal depth (two fit a compute unit), at least 40 stages, and
// a product is cut only when it is more than 1.3 times as deep: what a slice costs is its partial matrix, what it gains
// is the part of its depth by which a workgroup outlasts an even share of the call.  Preconditioning of ResNet-50-, VGG-16-
// (64 and 48 wide), small ResNet-50- (40 wide) shaped sets and two 1024-wide transformer blocks in ms: 0.996, 0.794, 0.492,
// 0.310, 1.190; slices of at most 150 stages of anything 1.5 times as deep as an even share of 400: 1.038, 0.863, 0.533, 0.319,
// 1.224; without slices: 0.990, 0.806, 0.534, 0.399, 1.192, and a 2048 x 1024 layer 0.230 instead of 0.147.  It loses where a
// call of 4 to 12 equal products fills one round of the chip as it is: eight 1025 x 1024 layers 0.286 sliced, 0.245 not.
constexpr int kMaxKSlices = 8;

int kslice_count(const GemmJob &j, long split_tiles, long cap)
{
    if (cap <= 0 || split_tiles >= 1024) return 1;     // enough tiles to keep every unit busy as it is
    if (j.mode != kStore || j.gate || j.wide_tiles) return 1;
    const long stages = (j.K + S_KT - 1) / S_KT;
    if (10 * stages <= 13 * cap) return 1;
    return (int)std::min<long>(kMaxKSlices, (stages + cap - 1) / cap);
}

// slices per job (1 = as it is); returns the floats of partial matrices needed
size_t plan_kslices(const GemmJob *jobs, int n, std::vector<int> &ks)
{
    ks.assign(n, 1);
    const bool wide = split_gemm_wide(jobs, n);
    long tiles = 0;
    double stages = 0.0;
    for (int i = 0; i < n; ++i)
        if (jobs[i].M > 0 && jobs[i].N > 0 && jobs[i].K > 0 && split_gemm_eligible(jobs[i], wide)) {
            const long t = (long)((jobs[i].M + S_BM - 1) / S_BM) * ((jobs[i].N + S_BN - 1) / S_BN);
            tiles += t;
            stages += (double)t * ((jobs[i].K + S_KT - 1) / S_KT);
        }
    const long least = tuning().gemm_kslice_stages;
    const long cap = least <= 0 ? 0 : std::max(least, (long)(stages / tuning().gemm_kslice_groups));
    size_t floats = 0;
    for (int i = 0; i < n; ++i) {
        if (!(jobs[i].M > 0 && jobs[i].N > 0 && jobs[i].K > 0) || !split_gemm_eligible(jobs[i], wide)) continue;
        ks[i] = kslice_count(jobs[i], tiles, cap);
        floats += (size_t)(ks[i] - 1) * align_up((size_t)jobs[i].M * jobs[i].N, 64);
    }
    return floats;
}

struct KRedProb {
    float *C;
    const float *P;      // first partial; the next ones follow at `stride` floats
    long ldc, stride;
    int M, N, parts;
    int blk_start;
};

struct KRedTable {
    int count;
    KRedProb p[kMaxProblems];
};

// C += P_1 + P_2 + ... (in this order); one thread per four consecutive entries of a row
__global__ __launch_bounds__(256) void gemm_kreduce_kernel(const KRedTable tab)
{
    int pi = 0;
    while (pi + 1 < tab.count && (int)blockIdx.x >= tab.p[pi + 1].blk_start) ++pi;
    const KRedProb &pr = tab.p[pi];
    const int n4 = (pr.N + 3) / 4;
    const long item = (long)(blockIdx.x - pr.blk_start) * 256 + threadIdx.x;
    if (item >= (long)pr.M * n4) return;
    const int m = (int)(item / n4), c0 = (int)(item - (long)m * n4) * 4;
    float *c = pr.C + (long)m * pr.ldc + c0;
    const float *q = pr.P + (long)m * pr.N + c0;
    const int cnt = min(4, pr.N - c0);
    float acc[4];
    for (int e = 0; e < cnt; ++e) acc[e] = c[e];
    for (int t = 0; t < pr.parts; ++t, q += pr.stride)
        for (int e = 0; e < cnt; ++e) acc[e] += q[e];
    for (int e = 0; e < cnt; ++e) c[e] = acc[e];
}

hipError_t gemm_launch_plain(const GemmJob *jobs, int n, hipStream_t s);
}  // namespace

hipError_t gemm_split_products(const GemmJob *jobs, int n, int cls, double definition, hipStream_t s)
{
    std::vector<int> idx(n);
    for (int i = 0; i < n; ++i) idx[i] = i;
    return split_gemm_launch(jobs, idx, s, cls, definition);
}

size_t gemm_workspace_bytes(const GemmJob *jobs, int n)
{
    std::vector<int> ks;
    return plan_kslices(jobs, n, ks) * sizeof(float);
}

hipError_t gemm_launch(const GemmJob *jobs, int n, hipStream_t s, void *work, size_t work_bytes)
{
    std::vector<int> ks;
    const size_t need = (work != nullptr) ? plan_kslices(jobs, n, ks) * sizeof(float) : 0;
    if (need == 0 || need > work_bytes) return gemm_launch_plain(jobs, n, s);
    std::vector<GemmJob> v;
    std::vector<KRedProb> red;
    float *part = static_cast<float *>(work);
    for (int i = 0; i < n; ++i) {
        const GemmJob &j = jobs[i];
        if (ks[i] <= 1) {
            v.push_back(j);
            continue;
        }
        const long stages = (j.K + S_KT - 1) / S_KT;
        const long per = (stages + ks[i] - 1) / ks[i] * S_KT;      // rows of K per slice
        const size_t stride = align_up((size_t)j.M * j.N, 64);
        int made = 0;
        for (long k0 = 0; k0 < j.K; k0 += per, ++made) {
            GemmJob t = j;
            t.A = j.A + k0 * j.lda;
            t.B = j.B + k0 * j.ldb;
            t.K = (int)std::min<long>(per, j.K - k0);
            t.wide_tiles = true;            // a slice stays on the split-bf16 kernel whatever its depth
            if (made > 0) {
                t.C = part + (size_t)(made - 1) * stride;
                t.ldc = j.N;
            }
            v.push_back(t);
        }
        KRedProb r;
        r.C = j.C; r.P = part; r.ldc = j.ldc; r.stride = (long)stride; r.M = j.M; r.N = j.N; r.parts = made - 1;
        r.blk_start = 0;
        if (r.parts > 0) red.push_back(r);
        part += (size_t)(ks[i] - 1) * stride;
    }
    hipError_t e = gemm_launch_plain(v.data(), (int)v.size(), s);
    if (e != hipSuccess) return e;
    for (size_t g0 = 0; g0 < red.size(); g0 += kMaxProblems) {
        KRedTable tab;
        tab.count = (int)std::min<size_t>(kMaxProblems, red.size() - g0);
        long blocks = 0;
        for (int k = 0; k < tab.count; ++k) {
            tab.p[k] = red[g0 + k];
            tab.p[k].blk_start = (int)blocks;
            blocks += ((long)tab.p[k].M * ((tab.p[k].N + 3) / 4) + 255) / 256;
        }
        KFAC_LAUNCH(KFAC_K_GEMM, s, gemm_kreduce_kernel, dim3((unsigned)blocks), dim3(256), 0, tab);
        timing_work(0.0, 0.0);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {
hipError_t gemm_launch_plain(const GemmJob *jobs, int n, hipStream_t s)
{
    if (n > 0 && jobs[0].chain) return chain_launch(jobs, n, s);
    const bool wide = split_gemm_wide(jobs, n);
    std::vector<int> cfg(n);
    std::vector<int> wave, split;
    for (int i = 0; i < n; ++i) {
        if (jobs[i].M > 0 && jobs[i].N > 0 && jobs[i].K > 0 && split_gemm_eligible(jobs[i], wide)) {
            cfg[i] = -1;
            split.push_back(i);
        } else if (jobs[i].M > 0 && jobs[i].N > 0 && jobs[i].K > 0 && wave_gemm_eligible(jobs[i])) {
            cfg[i] = -1;
            wave.push_back(i);
        } else {
            cfg[i] = choose_bm(jobs[i].M, jobs[i].N, jobs[i].mode == kSubLowerSkip);
        }
    }
    // A wave-unit workgroup owns 144 x 288 of a product and walks its whole depth at 110 us per 512 rows whatever else
    // the launch holds: a launch of few of them is nothing but that chain, which the 64-wide tiles spread over the chip
    // (eight products of the ResNet-50 shape, 129 x 512 at depth 512 the largest: 22 workgroups, 110 us; as 64-wide tiles 12
    // us more in a launch that is there anyway).
    long wave_blocks = 0;
    for (int i : wave) {
        const int mI = (jobs[i].M + W_MT - 1) / W_MT, nJ = (jobs[i].N + W_MT - 1) / W_MT;
        wave_blocks += jobs[i].mode == kSubLowerSkip ? (long)mI * (mI + 3) / 4 : (long)mI * ((nJ + 1) / 2);
    }
    if (!wave.empty() && wave_blocks < tuning().wave_gemm_min_blocks) {
        for (int i : wave) cfg[i] = choose_bm(jobs[i].M, jobs[i].N, jobs[i].mode == kSubLowerSkip);
        wave.clear();
    }
    {   // a small call is bound by its launches, not by its flops: one tile shape for all its products then
        double flops = 0.0, cost[4] = {0.0, 0.0, 0.0, 0.0};
        int used = 0;
        for (int i = 0; i < n; ++i) {
            const GemmJob &j = jobs[i];
            if (cfg[i] < 0 || j.mode == kSubLowerSkip) continue;      // the update products keep their own tile
            if (j.M <= 0 || j.N <= 0 || j.K <= 0) continue;
            used |= 1 << cfg[i];
            flops += 2.0 * j.M * j.N * j.K;
            for (int c = 0; c < 4; ++c) {
                const long bm = kBms[c];
                const long tm = (j.M + bm - 1) / bm, tn = (j.N + bm - 1) / bm;
                cost[c] += (double)tm * tn * bm * bm * (bm >= 128 ? 1.0 : (bm >= 64 ? 1.15 : 1.4)) * j.K;
            }
        }
        if (!tuning().gemm_bm && (used & (used - 1)) != 0 && flops < 8e9) {
            int best = 0;
            for (int c = 1; c < 4; ++c)
                if (cost[c] < cost[best]) best = c;
            for (int i = 0; i < n; ++i)
                if (cfg[i] >= 0 && jobs[i].mode != kSubLowerSkip) cfg[i] = best;
        }
    }
    if (!tuning().gemm_bm) {
        // a call whose block-tile products would not even give every CU a workgroup is bound by the K loop of one
        // tile: the 64-wide tiles spread it over four times as many CUs
        long wgs = 0;
        for (int i = 0; i < n; ++i) {
            const GemmJob &j = jobs[i];
            if (cfg[i] < 0 || j.mode == kSubLowerSkip || j.M <= 0 || j.N <= 0 || j.K <= 0) continue;
            const long bm = kBms[cfg[i]];
            wgs += ((j.M + bm - 1) / bm) * ((j.N + bm - 1) / bm);
        }
        if (wgs > 0 && wgs < 200)
            for (int i = 0; i < n; ++i)
                if (cfg[i] >= 0 && jobs[i].mode != kSubLowerSkip && kBms[cfg[i]] > 64) cfg[i] = 2;
    }
    // 32-bit offsets in the 64-wide kernel: operands of 2 GiB and more take the 128-wide tiles
    for (int i = 0; i < n; ++i)
        if (cfg[i] == 2 && ((long)jobs[i].K * jobs[i].lda * 4 > 0x7fffffffl || (long)jobs[i].K * jobs[i].ldb * 4 > 0x7fffffffl)) cfg[i] = 0;
    if (!split.empty()) {
        std::stable_sort(split.begin(), split.end(), [&](int a, int b) { return jobs[a].K > jobs[b].K; });
        hipError_t e = split_gemm_launch(jobs, split, s);
        if (e != hipSuccess) return e;
    }
    if (!wave.empty()) {
        // deepest products first: launches of similar depth, and the long workgroups start early
        std::stable_sort(wave.begin(), wave.end(), [&](int a, int b) { return jobs[a].K > jobs[b].K; });
        hipError_t e = wave_gemm_launch(jobs, wave, s);
        if (e != hipSuccess) return e;
    }
    for (int c = 0; c < 4; ++c) {
        GemmTable tab;
        tab.count = 0;
        int blocks = 0;
        auto flush = [&]() -> hipError_t {
            if (tab.count == 0) return hipSuccess;
            hipError_t e;
            switch (c) {
                case 0: e = launch_one<Tile<4, 2>>(tab, blocks, s); break;
                case 1: e = launch_one<Tile<3, 3>>(tab, blocks, s); break;
                case 2: e = launch_direct(tab, blocks, s); break;
                default: e = launch_one<Tile<1, 2>>(tab, blocks, s); break;
            }
            tab.count = 0;
            blocks = 0;
            return e;
        };
        for (int i = 0; i < n; ++i) {
            if (cfg[i] != c) continue;
            const GemmJob &j = jobs[i];
            if (j.M <= 0 || j.N <= 0 || j.K <= 0) continue;
            GemmProb &p = tab.p[tab.count++];
            const int bm = kBms[c];
            p.A = j.A; p.B = j.B; p.C = j.C;
            p.lda = j.lda; p.ldb = j.ldb; p.ldc = j.ldc;
            p.M = j.M; p.N = j.N; p.K = j.K;
            p.tm = (j.M + bm - 1) / bm;
            p.tn = (j.N + bm - 1) / bm;
            p.blk_start = blocks;
            tab.starts[tab.count - 1] = blocks;
            p.mode = j.mode;
            p.p0 = j.p0; p.p1 = j.p1; p.doff = j.doff;
            p.rv = j.rv; p.cv = j.cv; p.gamma = j.gamma; p.gate = j.gate; p.gate_cond = j.gate_cond;
            p.D = j.D; p.ldd = j.ldd;
            p.vecA = (((uintptr_t)j.A) % 16 == 0 && j.lda % 4 == 0) ? 1 : 0;
            p.vecB = (((uintptr_t)j.B) % 16 == 0 && j.ldb % 4 == 0) ? 1 : 0;
            blocks += (j.mode == kSubLowerSkip) ? p.tm * (p.tm + 1) / 2 : p.tm * p.tn;
            if (tab.count == kMaxGemmProblems) {
                hipError_t e = flush();
                if (e != hipSuccess) return e;
            }
        }
        hipError_t e = flush();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

}  // namespace kfac
