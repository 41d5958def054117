// Inverse of an SPD matrix of any but the smallest orders from its triangular factor, M + damping I = L L^T,
// (M + damping I)^-1 = X^T X with X = L^-1 (section 5.2 of the DP-KFAC paper names the Cholesky route; see invert.hip for the
// call).  Pivot blocks of 256, every product of their panels with a depth of up to the order of the matrix on the split-bf16
// core (split_common.hpp).
//
// Method.  L and X come row block by row block, from the left ("left-looking"): with block k = rows p0 .. p1 - 1 and
// W_m the 256 x n panel of an earlier block m (X's rows left of its diagonal block and in it, L^T's rows to the right),
//     V   = M[k, c] - sum_{m < k} W_m[:, k]^T W_m[:, c]     right of the diagonal block (c >= p1)
//     V   =         - sum_{m < k} W_m[:, k]^T W_m[:, c]     left of it (c < p0; W_m[:, c] is X's and begins at c's block)
//     W_k = X_kk V,   X_kk the inverse of the triangular factor of the diagonal block, after the same sum.
// A panel is stored as it is needed as an operand, depth first: rows p0 .. p1 - 1 of one n x n matrix T hold W_k.  Nothing is
// transposed, gathered or scattered, an entry of T is written once (once more by the product with X_kk, by the
// workgroup that holds it), and the elimination does 2/3 n^3 of the n^3 flops at a depth of up to n; the last third is
// X^T X, stored straight to both triangles of the result.
//
// Three launches per block whatever the number of matrices: the last panel's part of the next diagonal block
// (chol_next_kernel), its triangular inverse, a workgroup per matrix (chol_diag_kernel), everything else of the row
// block (chol_panel_kernel).  The diagonal block's sum over the panels before the last one runs with the panel launch
// of the block before.
//
// Orders 256 k + 1 (a bias column behind 256 k features): the last row by itself, two products of a matrix with a
// vector (chol_thin_kernel) instead of a block.
//
// Accuracy: sums right of the diagonal block start from M itself and go down from there: what a first panel takes away (the
// large eigenvalue of features that are not centred) is gone from the accumulator for the panels behind it.  Sums of
// the diagonal blocks and of X^T X start from zero, the latter with the last panel first: on matrices that their diagonal
// dominates, the large terms come last.
#pragma once

#include "split_common.hpp"

namespace kfac {

constexpr int CB = 256;                     // rows of a pivot block
constexpr int kMaxCholClasses = 64;         // distinct numbers of column tiles per launch
constexpr long kCholMaxOrder = 23000;       // operands stay below 2 GiB

struct CholProb {
    const float *M;      // lower triangle read
    float *T;            // working matrix [n + thin, ld]
    float *out;          // both triangles
    float *Xt;           // [256, 256] transposed inverse of the triangular factor of the diagonal block
    float *z;            // [n] workspace of the last row (thin)
    int *info;
    const float *dptr;   // device-side damping (overrides `damping` when not null)
    float damping;
    int n;               // order without the thin row
    int thin;            // 1: one more row and column behind it
    int ld, ldm, ldo;
};

constexpr int kCholUploadMax = 160;         // descriptors per upload launch

struct CholUpload {
    CholProb *dst;
    int count;
    CholProb p[kCholUploadMax];
};

struct CholClass {
    int first, count;    // matrices of the class in the table
    int nt;              // column tiles (of 128) of a matrix
    int per;             // workgroups per matrix in this launch
    int blk_start;       // first workgroup of the class (a multiple of 8)
};

struct CholSeq {
    const CholProb *tab;
    int nclass;
    int step;
    CholClass c[kMaxCholClasses];
};

__host__ __device__ __forceinline__ int chol_class_blocks(int count, int per) { return (count * per + 7) & ~7; }

// Workgroup -> (matrix, part).  Workgroup i runs on XCD i mod 8.  The matrices of a class up to a multiple of 8 are dealt
// to the XCDs, all workgroups of a matrix to one, matrix by matrix: they share its panels in that XCD's L2.  The up to 7
// left over are spread over all of them.
__device__ __forceinline__ bool chol_locate(const CholSeq &q, int &prob, int &part, int &nt)
{
    int ci = 0;
    while (ci + 1 < q.nclass && (int)blockIdx.x >= q.c[ci + 1].blk_start) ++ci;
    const CholClass &c = q.c[ci];
    const int full = c.count & ~7;
    int off = blockIdx.x - c.blk_start;
    nt = c.nt;
    if (off < full * c.per) {
        const int x = off & 7, i = off >> 3, m = i / c.per;
        prob = c.first + 8 * m + x;
        part = i - m * c.per;
        return true;
    }
    off -= full * c.per;
    const int m = off / c.per;
    if (m >= c.count - full) return false;
    prob = c.first + full + m;
    part = off - m * c.per;
    return true;
}

__global__ __launch_bounds__(64) void chol_upload_kernel(const CholUpload u)
{
    const int words = (int)(sizeof(CholProb) / 4);
    const unsigned *src = reinterpret_cast<const unsigned *>(u.p);
    unsigned *dst = reinterpret_cast<unsigned *>(u.dst);
    for (int e = threadIdx.x + blockIdx.x * 64; e < u.count * words; e += 64 * gridDim.x) dst[e] = src[e];
}

// ---- diagonal blocks -------------------------------------------------------------------------------------------------
// X of a diagonal block of up to 256 rows, a workgroup of 8 wavefronts.  The block lives in registers as 16 x 16 tiles of
// the MFMA result layout, tile (r, c) with wavefront (r mod 2, c mod 4), so that every step keeps all of them busy.  Step k:
// the rows of tile row k times X_kk, then the rank-16 update of the rows below (of X left of tile column k, of the symmetric
// rest right of the diagonal).  The operands of the first product are the tiles as they lie (the k of a 16 x 16 x 4 MFMA may
// come in any order); the new row goes through LDS, from where it is also stored.  The 16 pivots of the next X_kk run in one
// wavefront beside the update of the others.
// Bound: the fp32 MFMA of one CU (5440 of 16 x 16 x 4, 18 us at full rate) and the two barriers of a step.
constexpr int CD_WP = 260;                  // LDS pitch of a row of 256 (4 rows are 16 banks apart)
constexpr int CD_XP = 20;

// X of the 16 x 16 block in `src` (symmetric, pitch CD_XP) -> xs (row-major, zeros above the diagonal), one wavefront.
// Lane c < 16 holds column c of the block, lanes 16 .. 31 the columns of the identity.  A pivot that is not positive
// zeroes its row and is reported: 1-based place in the block, or 0.
__device__ __forceinline__ int chol_leaf(const float *src, float *xs, int lane)
{
    float col[16];
    const int c = lane & 15;
    {
        const floatx4 *p = reinterpret_cast<const floatx4 *>(src + c * CD_XP);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const floatx4 v = p[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) col[4 * i + e] = lane < 16 ? v[e] : (4 * i + e == c ? 1.f : 0.f);
        }
    }
    int fail = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(col[i]), i));
        const bool ok = d > 0.f;
        if (!ok && fail == 0) fail = i + 1;
        // 1 / sqrt(d): the instruction's last bit corrected; small pivots are scaled (it takes no denormal numbers)
        const bool tiny = d < 0x1p-96f;
        const float ds = tiny ? d * 0x1p64f : d;
        float r = __builtin_amdgcn_rsqf(ds);
        const float h = ds * r, e = __builtin_fmaf(-h, r, 1.f);
        r = __builtin_fmaf(0.5f * r, e, r);
        r = tiny ? r * 0x1p32f : r;
        r = ok && d <= 3.4028235e38f ? r : 0.f;
        const float w = col[i] * r;
        col[i] = w;
#pragma unroll
        for (int j = i + 1; j < 16; ++j) {
            const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j));
            col[j] = __builtin_fmaf(-s, w, col[j]);
        }
    }
    if (lane >= 16 && lane < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i) xs[i * CD_XP + c] = col[i];
    }
    return fail;
}

__global__ __launch_bounds__(512, 2) void chol_diag_kernel(const CholSeq q)
{
    __shared__ floatx4 ws4[16 * CD_WP / 4], xs4[16 * CD_XP / 4], leaf4[16 * CD_XP / 4];
    __shared__ int bad;
    float *ws = reinterpret_cast<float *>(ws4), *xs = reinterpret_cast<float *>(xs4), *leaf = reinterpret_cast<float *>(leaf4);
    const CholProb pr = q.tab[q.c[0].first + blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), a = w >> 2, b = w & 3;      // tile rows a, a + 2, ..., tile columns b, b + 4, ...
    const int lq = lane >> 4, ln = lane & 15;
    const int p0 = q.step * CB, bs = min(CB, pr.n - p0), nb = (bs + 15) >> 4;
    const bool panel = pr.n > CB;
    if (tid == 0) bad = 0;

    floatx4 acc[8][4];
    {   // tile (r, c), c >= r: element (16 r + 4 lq + v, 16 c + ln) of the upper triangle, from the lower one
        const float *S = q.step == 0 ? pr.M : pr.T + (long)p0 * pr.ld + p0;
        const long lds = q.step == 0 ? pr.ldm : pr.ld;
        const float damping = q.step == 0 ? (pr.dptr ? *pr.dptr : pr.damping) : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * (2 * i + a) + 4 * lq, c = 16 * (4 * j + b) + ln;
                floatx4 v = {0.f, 0.f, 0.f, 0.f};
                if (c < bs && r <= c) {
                    const float *p = S + c * lds + r;
                    if (r + 3 <= c) {
                        typedef float uf4 __attribute__((ext_vector_type(4), aligned(4)));
                        v = *reinterpret_cast<const uf4 *>(p);
                    } else {
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            if (r + e <= c) v[e] = p[e];
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (r + e == c) v[e] = c < bs ? v[e] + damping : 1.f;      // rows past the edge: the identity
                acc[i][j] = v;
                if (j == 3) __builtin_amdgcn_sched_barrier(0);
            }
    }
    // Step k forms row k; step -1 only inverts the first diagonal tile.
    for (int k = -1;; ++k) {
        __syncthreads();
        if (k >= 0) {
            // the new row: X_kk times the tiles of tile row k
            if (a == (k & 1)) {
                const floatx4 x = *reinterpret_cast<const floatx4 *>(xs + ln * CD_XP + 4 * lq);
                floatx4 row[4];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (i == (k >> 1)) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) row[j] = acc[i][j];
                    }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int c = 4 * j + b;
                    floatx4 t = {0.f, 0.f, 0.f, 0.f};
                    if (c == k) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) t[v] = xs[(4 * lq + v) * CD_XP + ln];
                    } else {
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) t = __builtin_amdgcn_mfma_f32_16x16x4f32(x[jj], row[j][jj], t, 0, 0, 0);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) ws[(4 * lq + v) * CD_WP + 16 * c + ln] = t[v];
                    // X^T, from where the panel product reads X
                    if (panel) *reinterpret_cast<floatx4 *>(pr.Xt + (16 * c + ln) * CB + 16 * k + 4 * lq) = c <= k ? t : floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {   // rows w, w + 8 of the new row of X, zeros right of the diagonal
                const int row = 16 * k + w + 8 * u, c = 4 * lane;
                if (row < bs && p0 + c < pr.ld) {
                    const floatx4 v = *reinterpret_cast<const floatx4 *>(ws + (w + 8 * u) * CD_WP + c);
                    *reinterpret_cast<floatx4 *>(pr.T + (long)(p0 + row) * pr.ld + p0 + c) = c < 16 * (k + 1) ? v : floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
            if (k + 1 == nb) break;
        }
        if (a == ((k + 1) & 1) && b == ((k + 1) & 3)) {
            // the tile that the next step begins with ahead of all others; through LDS, mirrored
            floatx4 t;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i == ((k + 1) >> 1)) {
                    t = acc[i][i >> 1];
                    if (k >= 0) {
                        float f[4];
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) f[jj] = ws[(4 * lq + jj) * CD_WP + 16 * (k + 1) + ln];
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) t = __builtin_amdgcn_mfma_f32_16x16x4f32(-f[jj], f[jj], t, 0, 0, 0);
                    }
                }
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * lq + v <= ln) {
                    leaf[(4 * lq + v) * CD_XP + ln] = t[v];
                    leaf[ln * CD_XP + 4 * lq + v] = t[v];
                }
            const int f = chol_leaf(leaf, xs, lane);
            if (lane == 0 && f != 0 && bad == 0) bad = 16 * (k + 1) + f;
        }
        if (k < 0) continue;
        __builtin_amdgcn_sched_barrier(0);
        float br[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) br[j][jj] = ws[(4 * lq + jj) * CD_WP + 16 * (4 * j + b) + ln];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 2 * i + a;
            if (r <= k) continue;
            float ar[4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) ar[jj] = -ws[(4 * lq + jj) * CD_WP + 16 * r + ln];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = 4 * j + b;
                if (c > k && c < r) continue;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[jj], br[j][jj], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (tid == 0) {
        if (q.step == 0) *pr.info = bad;
        else if (bad != 0 && *pr.info == 0) *pr.info = p0 + bad;
    }
}

// Diagonal block k + 1 (lower triangle) -= W_k[:, block]^T W_k[:, block]: 32 x 32 tiles, a wavefront each, on the split
// arithmetic.  Operands go straight from memory to the wavefront that cuts them, four stages of 16 rows in flight; no LDS, no
// barrier.  A launch of five blocks: 14 us.
__global__ __launch_bounds__(64) void chol_next_kernel(const CholSeq q)
{
    int prob, part, nt;
    if (!chol_locate(q, prob, part, nt)) return;
    const CholProb pr = q.tab[prob];
    int bi, bj;
    tri_decode(part, bi, bj);
    const int p0 = q.step * CB, q0 = p0 + CB, bn = min(CB, pr.n - q0);
    const int m0 = 32 * bi, n0 = 32 * bj, nst = CB / 16;
    if (m0 >= bn) return;
    const int lane = threadIdx.x, lr = lane & 31, lg = lane >> 5;
    const unsigned pitch = (unsigned)pr.ld * 4u;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(pr.T + (long)p0 * pr.ld + q0, 0, (int)(CB * pitch - 4u * (unsigned)q0), 0x00020000);
    // columns past the edge repeat the last one: their results are not stored
    const unsigned ao = (unsigned)min(m0 + lr, bn - 1) * 4u + 8u * (unsigned)lg * pitch, bo = (unsigned)min(n0 + lr, bn - 1) * 4u + 8u * (unsigned)lg * pitch;
    float x[4][8], y[4][8];                   // rows 16 g + 8 lg + e
    auto load = [&](int set, int g) {
        const int gg = min(g, nst - 1);       // past the end: the last stage again, not used
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[set][e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, ao, (unsigned)(16 * gg + e) * pitch, 0));
            y[set][e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, bo, (unsigned)(16 * gg + e) * pitch, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pieces = [&](sbf16x8 (&f)[3], const float (&v)[8]) {
        float x0[4] = {v[0], v[1], v[2], v[3]}, x1[4] = {v[4], v[5], v[6], v[7]};
        SplitCut k0, k1;
        k0.scale(x0); k1.scale(x1);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            k0.half(x0, 0, 4); k1.half(x1, 0, 4);
            const suint2 u = k0.pack(), t = k1.pack();
            f[p] = __builtin_bit_cast(sbf16x8, suint4{u.x, u.y, t.x, t.y});
            k0.top(0, 4); k1.top(0, 4);
            k0.rest(x0, 0, 4); k1.rest(x1, 0, 4);
        }
        const suint2 u = k0.pack_last(x0), t = k1.pack_last(x1);
        f[2] = __builtin_bit_cast(sbf16x8, suint4{u.x, u.y, t.x, t.y});
    };
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) load(t, t);
    sbf16x8 A[2][3], B[2][3];
    pieces(A[0], x[0]);
    pieces(B[0], y[0]);
    load(0, 4);
    for (int g = 0; g < nst; g += 4)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // the cut of the next stage between the products of this one, which wait for each other
            pieces(A[(t + 1) & 1], x[(t + 1) & 3]);
            pieces(B[(t + 1) & 1], y[(t + 1) & 3]);
            constexpr int pieceA[6] = {2, 1, 1, 0, 0, 0}, pieceB[6] = {0, 1, 0, 2, 1, 0};
#pragma unroll
            for (int m = 0; m < 6; ++m) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t & 1][pieceA[m]], B[t & 1][pieceB[m]], acc, 0, 0, 0);
#pragma unroll
            for (int m = 0; m < 6; ++m) {
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
        const unsigned ca = ao - 8u * (unsigned)lg * pitch, cb = bo - 8u * (unsigned)lg * pitch;
        for (int k = 0; k < 16 * nst; k += 2) {
            const float u = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, ca + (unsigned)(k + lg) * pitch, 0, 0));
            const float v = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, cb + (unsigned)(k + lg) * pitch, 0, 0));
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u, v, acc, 0, 0, 0);
        }
    }
    const int n = n0 + lr;
    float *C = pr.T + (long)q0 * pr.ld + q0;
    float old[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + 8 * (v >> 2) + 4 * lg + (v & 3);
        old[v] = m < bn && n <= m ? C[(long)m * pr.ld + n] : 0.f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + 8 * (v >> 2) + 4 * lg + (v & 3);
        if (m < bn && n <= m) C[(long)m * pr.ld + n] = __builtin_fmaf(-unscale, acc[v], old[v]);
    }
}

// ---- panels ----------------------------------------------------------------------------------------------------------
__host__ __device__ __forceinline__ int chol_panel_parts(int nt, int k)
{
    const int right = nt - 2 * (k + 1) > 0 ? nt - 2 * (k + 1) : 0;
    return right + 2 * k + (right < 2 ? right : 2);
}

// Operands of a tile: rows of T from row `row` on (K of them), columns ca .. of A, cb .. of B; B from another matrix
// where `b` is given.
__device__ __forceinline__ void chol_source(SplitSrc<kRows> &src, const float *A, int lda, int ca, int arows, const float *B, int ldb, int cb, int bcols, int K, int tid)
{
    src.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(A), 0, (int)((long)K * lda * 4), 0x00020000);
    src.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(B), 0, (int)((long)K * ldb * 4), 0x00020000);
    src.lda4 = (unsigned)lda * 4u;
    src.ldb4 = (unsigned)ldb * 4u;
    src.nstages = (K + S_KT - 1) / S_KT;
    src.init_thread(tid);
    src.lim_a = arows;
    src.lim_b = bcols;
    src.va[0] = src.col_a(0) < arows ? (unsigned)(ca + src.col_a(0)) * 4u + 4u * (unsigned)src.kq * src.lda4 : W_OOB;
    src.vb[0] = src.col_b(0) < bcols ? (unsigned)(cb + src.col_b(0)) * 4u + 4u * (unsigned)src.kq * src.ldb4 : W_OOB;
}

// Row block k: a tile of 256 rows and 128 columns per workgroup, sum over the panels before it, then, in the same
// accumulators, X_kk times the tile (which passes through its place in T: written and read back by the same
// workgroup).  Parts of a matrix, longest first: the tiles right of the diagonal block, those left of it (their depth
// begins at their columns' block), the diagonal block after this one (sum alone; all panels but W_k).
__global__ __launch_bounds__(256, 2) void chol_panel_kernel(const CholSeq q)
{
    __shared__ SplitLds L;
    int prob, part, nt;
    if (!chol_locate(q, prob, part, nt)) return;
    const CholProb pr = q.tab[prob];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
    int lr = lane & 31, lg = lane >> 5;
    const int k = q.step, n = pr.n, ld = pr.ld, p0 = k * CB, bs = min(CB, n - p0), p1 = p0 + bs;
    const int right = max(0, nt - 2 * (k + 1));
    const bool is_right = part < right, is_diag = part >= right + 2 * k;
    const int c0 = is_right ? p1 + S_BN * part : is_diag ? p1 + S_BN * (part - right - 2 * k) : S_BN * (part - right);
    const int kbeg = is_right || is_diag ? 0 : c0 & ~(CB - 1);
    const int r0 = is_diag ? p1 : p0, nrows = is_diag ? min(CB, n - p1) : bs;
    const int ncols = min(S_BN, (is_right || is_diag ? n : p0) - c0);
    const int mleft = nrows - wm * (S_BM / 2);
    const int rows = mleft <= 0 || wn * 64 >= ncols ? 0 : (mleft + 31) / 32;

    // element (m, n) of the part of M above the diagonal, from below it: m and the three rows after it are neighbours there
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.M + (long)c0 * pr.ldm + r0), 0, (int)((long)(ncols - 1) * pr.ldm * 4 + 4 * CB), 0x00020000);
    auto from_m = [&](int ti, int tj, int g) {
        const int m = wm * (S_BM / 2) + ti * 32 + 8 * g + 4 * lg, c = wn * 64 + tj * 32 + lr;
        return __builtin_bit_cast(sint4, __builtin_amdgcn_raw_buffer_load_b128(rm, c < ncols ? (unsigned)(c * pr.ldm + m) * 4u : W_OOB, 0, 0));
    };
    bool first = true;
    auto init = [&](floatx16 (&acc)[8], float unit) {
        if (first && is_right) {
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
#pragma unroll
                for (int tj = 0; tj < 2; ++tj)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const sint4 v = from_m(ti, tj, g);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[ti * 2 + tj][4 * g + e] = -unit * __int_as_float(v[e]);
                        if (tj == 1 && g == 3) __builtin_amdgcn_sched_barrier(0);
                    }
        } else {
            SplitZero()(acc, unit);
        }
    };
    SplitSrc<kRows> src;
    const float *rowk = pr.T + (long)p0 * ld;
    constexpr int EP = 68;                                   // LDS row pitch of a chunk (floats)
    float *wl = reinterpret_cast<float *>(L.ring) + w * 32 * EP;
    int rr = lane >> 4, c4 = (lane & 15) * 4;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        // (or the addresses of both passes are computed ahead of the loop and kept in scratch memory)
        asm volatile("" : "+v"(lr), "+v"(lg), "+v"(rr), "+v"(c4));
        if (pass == 0) chol_source(src, pr.T + (long)kbeg * ld, ld, r0, nrows, pr.T + (long)kbeg * ld, ld, c0, ncols, p0 - kbeg, tid);
        else chol_source(src, pr.Xt, CB, 0, nrows, rowk, ld, c0, ncols, bs, tid);
        first = pass == 0;
        floatx16 acc[8];
        float none[4];
        const float unscale = split_tile<kRows, false, false>(src, L, acc, none, 0, rows, wm, wn, tid, init);
        if (is_diag) {
            // lower triangle, as the kernels of the diagonal blocks read it: M + damping I minus the sum
            if (rows == 0) return;
            const float damping = pr.dptr ? *pr.dptr : pr.damping;
            const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(pr.T + (long)r0 * ld + r0, 0, (int)((long)nrows * ld * 4 - 4l * r0), 0x00020000);
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
#pragma unroll
                for (int tj = 0; tj < 2; ++tj) {
                    const int cm = wn * 64 + tj * 32 + lr, c = c0 - r0 + cm;     // column of the block = row of its lower triangle
                    sint4 old[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int m = wm * (S_BM / 2) + ti * 32 + 8 * g + 4 * lg;
                        const unsigned o = (unsigned)(cm * pr.ldm + m) * 4u;
                        const bool in = c < nrows && m <= c;
                        old[g] = __builtin_bit_cast(sint4, __builtin_amdgcn_raw_buffer_load_b128(rm, in && m + 3 <= c ? o : W_OOB, 0, 0));
                        if (__any(in && m + 3 > c)) {
#pragma unroll
                            for (int e = 0; e < 3; ++e) {
                                const int x = __builtin_amdgcn_raw_buffer_load_b32(rm, in && m + 3 > c && m + e <= c ? o + 4u * (unsigned)e : W_OOB, 0, 0);
                                if (m + 3 > c) old[g][e] = x;
                            }
                        }
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int m = wm * (S_BM / 2) + ti * 32 + 8 * g + 4 * lg;
                        const unsigned o = (unsigned)(c * ld + m) * 4u;
                        const bool in = c < nrows && m <= c;
                        floatx4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e] = __builtin_fmaf(-unscale, acc[ti * 2 + tj][4 * g + e], __int_as_float(old[g][e]) + (m + e == c ? damping : 0.f));
                        // (what lies right of the diagonal is not read: a lane's four columns are stored whole, ld is a multiple of 4)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(suint4, v), rt, in ? o : W_OOB, 0, 0);
                    }
                }
            return;
        }
        // (see gemm_split_kernel: through LDS, 16 lanes along a row; all loads of a batch ahead of its stores)
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(rowk), 0, (int)((long)bs * ld * 4), 0x00020000);
        const float sign = pass == 0 ? -unscale : unscale;
        const int col = c0 + wn * 64 + c4;
        const bool live = wn * 64 + c4 < ncols;              // the pitch is a multiple of 4: a lane's columns exist or do not
        if (rows > 0) {
#pragma unroll
            for (int ti = 0; ti < 4; ++ti) {
#pragma unroll
                for (int tj = 0; tj < 2; ++tj)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        wl[(8 * (v >> 2) + 4 * lg + (v & 3)) * EP + tj * 32 + lr] = acc[ti * 2 + tj][v] * sign;
                // (LDS operations of one wavefront complete in order: no barrier between these writes and the reads)
#pragma unroll
                for (int g = 0; g < 8; ++g) {
                    const int m = wm * (S_BM / 2) + ti * 32 + 4 * g + rr;
                    const floatx4 val = *reinterpret_cast<const floatx4 *>(wl + (4 * g + rr) * EP + c4);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(suint4, val), rc, live && m < bs ? (unsigned)(m * ld + col) * 4u : W_OOB, 0, 0);
                }
            }
        }
        __syncthreads();                                     // the stores of the workgroup are done, its chunks free
    }
}

// ---- the last row of orders 256 k + 1 --------------------------------------------------------------------------------
// z = X m for the last row m of M (without its corner): a wavefront per row of X
__global__ __launch_bounds__(256) void chol_thin_z_kernel(const CholSeq q)
{
    int prob, part, nt;
    if (!chol_locate(q, prob, part, nt)) return;
    const CholProb pr = q.tab[prob];
    if (!pr.thin) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const float *m = pr.M + (long)pr.n * pr.ldm;
    // rows 4 w .. 4 w + 3 of the 16 of this workgroup: all end in the same 256 columns, zeros right of the diagonal
    const int i0 = 16 * part + 4 * w;
    if (i0 >= pr.n) return;
    const int end = (i0 & ~(CB - 1)) + CB;               // n is a multiple of 256
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float *row = pr.T + (long)i0 * pr.ld;
    for (int j = 4 * lane; j < end; j += 256) {
        const floatx4 x0 = *reinterpret_cast<const floatx4 *>(row + j), x1 = *reinterpret_cast<const floatx4 *>(row + pr.ld + j),
                      x2 = *reinterpret_cast<const floatx4 *>(row + 2l * pr.ld + j), x3 = *reinterpret_cast<const floatx4 *>(row + 3l * pr.ld + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float b = m[j + e];
            acc[0] = __builtin_fmaf(x0[e], b, acc[0]);
            acc[1] = __builtin_fmaf(x1[e], b, acc[1]);
            acc[2] = __builtin_fmaf(x2[e], b, acc[2]);
            acc[3] = __builtin_fmaf(x3[e], b, acc[3]);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float s = acc[r];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) pr.z[i0 + r] = s;
    }
}

// s = c + damping - z^T z, x = 1 / sqrt(s), last row of X: -x z^T X and x; last row and column of the inverse: x times that
__global__ __launch_bounds__(1024) void chol_thin_row_kernel(const CholSeq q)
{
    __shared__ float part_s[16], part_y[16][64];
    int prob, part, nt;
    if (!chol_locate(q, prob, part, nt)) return;
    const CholProb pr = q.tab[prob];
    if (!pr.thin) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n = pr.n;
    const int j0 = 64 * part;
    if (j0 >= n) return;
    float s = 0.f;
    for (int i = tid; i < n; i += 1024) s = __builtin_fmaf(pr.z[i], pr.z[i], s);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) part_s[w] = s;
    // column j0 + lane of X from its diagonal block down, rows w, w + 16, ...
    float y = 0.f;
    const float *col = pr.T + j0 + lane;
    for (int i = (j0 & ~(CB - 1)) + w; i < n; i += 128) {
        float x[8], z[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = min(i + 16 * u, n - 1);
            x[u] = col[(long)r * pr.ld];
            z[u] = i + 16 * u < n ? pr.z[r] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) y = __builtin_fmaf(x[u], z[u], y);
    }
    part_y[w][lane] = y;
    __syncthreads();
    if (w != 0) return;
    s = 0.f;
    y = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) { s += part_s[i]; y += part_y[i][lane]; }
    const float damping = pr.dptr ? *pr.dptr : pr.damping;
    const float d = pr.M[(long)n * pr.ldm + n] + damping - s;
    const bool ok = d > 0.f;
    const float x = ok ? 1.f / sqrtf(d) : 0.f, xi = -x * y;
    pr.T[(long)n * pr.ld + j0 + lane] = xi;
    pr.out[(long)n * pr.ldo + j0 + lane] = x * xi;
    pr.out[(long)(j0 + lane) * pr.ldo + n] = x * xi;
    if (part == 0 && lane == 0) {
        if (!ok && *pr.info == 0) *pr.info = n + 1;
        pr.T[(long)n * pr.ld + n] = x;
        pr.out[(long)n * pr.ldo + n] = x * x;
    }
}

// ---- the inverse -----------------------------------------------------------------------------------------------------
// 256 x 128 tiles of X^T X that reach the lower triangle, tile row by tile row: those of the first rows are the deepest
__host__ __device__ __forceinline__ int chol_out_parts(int nt)
{
    int c = 0;
    for (int i = 0; 2 * i < nt; ++i) c += 2 * i + 2 < nt ? 2 * i + 2 : nt;
    return c;
}

__global__ __launch_bounds__(256, 2) void chol_out_kernel(const CholSeq q)
{
    __shared__ SplitLds L;
    int prob, part, nt;
    if (!chol_locate(q, prob, part, nt)) return;
    const CholProb pr = q.tab[prob];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
    const int lr = lane & 31, lg = lane >> 5;
    int I = 0;
    for (;; ++I) {
        const int c = min(2 * I + 2, nt);
        if (part < c) break;
        part -= c;
    }
    const int m0 = S_BM * I, n0 = S_BN * part, n = pr.n, full = n + pr.thin;
    const int nrows = min(S_BM, n - m0), ncols = min(S_BN, n - n0);
    const int mleft = nrows - wm * (S_BM / 2);
    // a wavefront wholly above the diagonal has nothing to compute
    const int rows = mleft <= 0 || wn * 64 >= ncols || n0 + wn * 64 > m0 + wm * (S_BM / 2) + S_BM / 2 - 1 ? 0 : (mleft + 31) / 32;
    SplitSrc<kRows> src;
    const float *X = pr.T + (long)m0 * pr.ld;
    chol_source(src, X, pr.ld, m0, nrows, X, pr.ld, n0, ncols, full - m0, tid);
    src.down = true;
    floatx16 acc[8];
    float none[4];
    const float unscale = split_tile<kRows, false, false>(src, L, acc, none, 0, rows, wm, wn, tid);
    if (rows == 0) return;
    const int ldo = pr.ldo, mw = m0 + wm * (S_BM / 2), nw = n0 + wn * 64;
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(pr.out, 0, (int)((long)full * ldo * 4), 0x00020000);
    // the mirror image, straight from the accumulators: a lane's four rows are neighbours there
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int m = mw + ti * 32 + 8 * g + 4 * lg, c = nw + tj * 32 + lr;
                floatx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[ti * 2 + tj][4 * g + e] *= unscale;
                const unsigned o = (unsigned)(c * ldo + m) * 4u;
                const bool all = c < m && m + 3 < n;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(suint4, v), rc, all ? o : W_OOB, 0, 0);
                if (__any(!all && c < m + 3 && m < n && c < n)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[e]), rc, !all && c < m + e && m + e < n ? o + 4u * (unsigned)e : W_OOB, 0, 0);
                }
            }
    constexpr int EP = 68;
    float *wl = reinterpret_cast<float *>(L.ring) + w * 32 * EP;
    const int rr = lane >> 4, c4 = (lane & 15) * 4;
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int v = 0; v < 16; ++v) wl[(8 * (v >> 2) + 4 * lg + (v & 3)) * EP + tj * 32 + lr] = acc[ti * 2 + tj][v];
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int m = mw + ti * 32 + 4 * g + rr, c = nw + c4;
            const floatx4 val = *reinterpret_cast<const floatx4 *>(wl + (4 * g + rr) * EP + c4);
            const int have = m < n ? m + 1 - c : 0;          // columns up to the diagonal
            const unsigned o = (unsigned)(m * ldo + c) * 4u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(suint4, val), rc, have >= 4 ? o : W_OOB, 0, 0);
            if (__any(have > 0 && have < 4)) {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[e]), rc, have < 4 && e < have ? o + 4u * (unsigned)e : W_OOB, 0, 0);
            }
        }
    }
}

}  // namespace kfac
