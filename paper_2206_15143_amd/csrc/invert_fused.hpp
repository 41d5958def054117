// One-launch-per-step form of the blocked symmetric sweep (see invert.hip for
// the method), for the small and medium factors where the three-kernel step
// (pivot, panel, update) is bound by launch latency and by the serial pivot
// block inversion rather than by flops.
//
// Step K of the sweep is ONE launch over all lower-triangular 64 x 64 tiles of
// all matrices that are still active:
//   - a tile in the pivot row/column (panel tile) computes W = V P and stores
//     it in place;
//   - any other tile (i, j) loads V_i and V_j, forms W_i = V_i P on the MFMA
//     units again (cheaper than a launch that would share it) and applies
//     M_ij -= W_i V_j^T;
//   - tiles in row/column K+1 also store their new values K-major into the
//     side buffer V' that step K+1 reads (so the panel is never read from the
//     matrix while panel tiles overwrite it);
//   - the workgroup of tile (K+1, K+1) goes on to invert that block, which is
//     final for step K+1 once updated: P' and the in-place block are ready
//     when the launch ends.  That tile gets block index 0 of its matrix so
//     that it starts first.
// Step 0 reads the input factor (plus damping) instead of the working matrix and
// the last step of a matrix stores the negated result to both triangles, so
// there is no initialisation or finishing pass.
// P and V are double buffered by step parity.  Problem descriptors live in
// device memory (uploaded by a small kernel from kernel arguments), so one
// launch covers any number of matrices; the launch argument only carries the
// table of distinct sizes.
#pragma once

#include "tn_engine.hpp"

namespace kfac {

constexpr int FNB = 64;            // pivot block order
constexpr int kMaxInvClasses = 24; // distinct numbers of pivot blocks per launch sequence

struct InvProbF {
    const float *M;   // input factor [n, n], lower triangle read
    float *W;         // working matrix = output [n, n]
    float *P;         // 2 x [64, 64] pivot-block inverses (step parity)
    float *Vt;        // 2 x [64, ldv] K-major panels (step parity)
    float *S;         // 2 x [64, 64] pivot blocks before their inversion, both triangles (step parity)
    int *gate;        // 2 flags (step parity): the pivot block is ill-conditioned, refine the panel product;
                      // a third that stays set once either was (read by the bordering of orders 64 k + 1)
    int *info;
    int n;
    int ldv;          // n rounded up to 4
    float damping;
    int nblk;
    int ldm, ldw;     // row pitches of M and W
    const float *dptr; // device-side damping (overrides `damping` when not null)
    int border;        // one more row and column behind the order n = 64, bordered by the workgroup that inverts the block:
                       // 2 with the refinement step, 1 with it where the block is ill-conditioned (see invert.hip); 0: none
};

// The same with pointers that are known to point to device memory.  Of a pointer read from memory the compiler cannot
// tell: it uses flat accesses, which count as LDS accesses too and make every wait for LDS one for all of memory.
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) int gint;
typedef __attribute__((address_space(1))) floatx4 gfloatx4;
typedef float ufloatx4 __attribute__((ext_vector_type(4), aligned(4)));    // rows of a matrix of any order
typedef __attribute__((address_space(1))) ufloatx4 gufloatx4;
struct InvProbG {
    const gfloat *M;
    gfloat *W, *P, *Vt, *S;
    gint *gate, *info;
    const gfloat *dptr;
    int n, ldv, nblk, ldm, ldw;
    float damping;
    int border;
};
__device__ __forceinline__ InvProbG load_prob(const InvProbF &p)
{
    return InvProbG{(const gfloat *)p.M, (gfloat *)p.W, (gfloat *)p.P, (gfloat *)p.Vt, (gfloat *)p.S, (gint *)p.gate,
                    (gint *)p.info, (const gfloat *)p.dptr, p.n, p.ldv, p.nblk, p.ldm, p.ldw, p.damping, p.border};
}

constexpr int kInvUploadMax = 224;   // descriptors per upload launch (a 22 KB kernel argument)

struct InvUpload {
    InvProbF *dst;
    int count;
    InvProbF p[kInvUploadMax];
};

struct InvClass {
    int first;       // index of the first problem of this class in the device table
    int count;       // problems in the class
    int nblk;
    int per;         // blocks per problem in this launch
    int blk_start;   // first block of the class in this launch (a multiple of 8)
};

struct InvSeq {
    const InvProbF *tab;
    int nclass;
    int step;
    int heads;           // blocks ahead of the first class: block 0 of every matrix, rounded up to a multiple of 8
    int nprob;           // matrices in this launch
    float refine_cond;   // panel products of pivot blocks whose condition number exceeds this are refined (< 0: never)
    InvClass c[kMaxInvClasses];
};

// The descriptors of a call of few matrices, as an argument of its first kernel, which leaves them in the device table for
// the later ones: no launch ahead of it (6 us of every outer step of the blocked sweep, whose pivot blocks come this way).
template <int N>
struct InvInline {
    InvProbF p[N];
};

__global__ __launch_bounds__(64) void inv_upload_kernel(const InvUpload u)
{
    // plain vector stores of the descriptors into the device table
    const int words = (int)(sizeof(InvProbF) / 4);
    const unsigned *src = reinterpret_cast<const unsigned *>(u.p);
    unsigned *dst = reinterpret_cast<unsigned *>(u.dst);
    for (int e = threadIdx.x + blockIdx.x * 64; e < u.count * words; e += 64 * gridDim.x) dst[e] = src[e];
}

// Block -> (matrix, block of that matrix).  The first q.heads blocks are block 0 of every matrix, the one that goes
// on to invert the next pivot block: dispatched first, that chain runs beside the other tiles.  The blocks 1 .. per - 1
// follow class by class (a class: matrices with the same number of pivot blocks, whatever their order).  Inside a
// class the matrices of the largest multiple of 8 are dealt block-major, block `local` of every matrix before block
// `local + 1` of any: workgroup i runs on XCD i mod 8, so every block of a matrix runs on the same XCD and its panels
// and pivot inverse are fetched into one L2 instead of eight.  The up to 7 matrices left over are dealt the same way
// among themselves, so that their blocks are spread over all XCDs (rounded up to slots of 8 they ran on the first
// XCDs alone: a network with 107 different layer shapes, most of them once, kept one XCD busy and seven idle; the
// fused class of that network took 14.2 ms of kernel time, now 9.2 ms).
__host__ __device__ __forceinline__ int seq_class_blocks(int count, int per)
{
    return per > 1 ? (count * (per - 1) + 7) & ~7 : 0;
}

__device__ __forceinline__ bool seq_locate(const InvSeq &q, int blk, int &prob, int &local)
{
    if (blk < q.heads) {
        prob = q.c[0].first + blk;       // the matrices of a sequence are neighbours in the table
        local = 0;
        return blk < q.nprob;
    }
    int ci = 0;
    while (ci + 1 < q.nclass && blk >= q.c[ci + 1].blk_start) ++ci;
    const InvClass &c = q.c[ci];
    const int full = c.count & ~7, rest = c.count - full, each = c.per - 1;
    int off = blk - c.blk_start;
    if (off < full * each) {
        local = off / full;
        prob = c.first + off - local * full;
    } else {
        off -= full * each;
        if (off >= rest * each) return false;
        local = off / rest;
        prob = c.first + full + off - local * rest;
    }
    ++local;
    return true;
}

// One pivot of the in-register 16 x 16 sweep (see sweep64_blocked): lane (lr, lk) holds D[lr][4lk..4lk+3].
template <int K>
__device__ __forceinline__ void sweep16_pivot(float (&d)[4], int lr, int lk, int c0, int &fail)
{
    float rk[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
        rk[m] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(d[m]), 0x150 + K, 0xf, 0xf, false));
    // the pivot D[K][K] sits in lane K + 16*(K>>2), register K & 3
    const float p = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d[K & 3]), K + 16 * (K >> 2)));
    if (!(p > 0.f) && fail == 0) fail = c0 + K + 1;
    const float ip = __builtin_amdgcn_rcpf(p);   // 1 ulp reciprocal: far below the fp32 error of the sweep
    // column element D[i][K] = D[K][i]: element i of the row, held by lane i + 16*(i>>2) in register i & 3.  (The column itself, equal
    // up to rounding, would come without the LDS round trip of a bpermute; at a condition of 1e5 the error was 0.4 then.)
    float mine = rk[0];
    mine = (lr & 3) == 1 ? rk[1] : mine;
    mine = (lr & 3) == 2 ? rk[2] : mine;
    mine = (lr & 3) == 3 ? rk[3] : mine;
    const float ci = __int_as_float(__builtin_amdgcn_ds_bpermute((lr + 16 * (lr >> 2)) * 4, __float_as_int(mine)));
    const float cip = ci * ip;
    const bool prow = (lr == K);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const float upd = __builtin_fmaf(-cip, rk[m], d[m]);
        const float onr = rk[m] * ip;
        float v = prow ? onr : upd;
        if (m == (K & 3)) v = (lk == (K >> 2)) ? (prow ? -ip : cip) : v;
        d[m] = v;
    }
}

// Sweep of a 64 x 64 pivot block held in LDS (full symmetric storage, row pitch
// SW_PITCH; blocks smaller than 64 are padded with the identity by the caller).  Four sub-steps of 16
// pivots.  Per sub-step: wavefront 0 sweeps the 16 x 16 pivot block inside its registers (lane (i, q)
// holds D[i][4q..4q+3]; the pivot row reaches the lanes by DPP row broadcast, the pivot column, equal to
// the row by symmetry, by one ds_bpermute: no barrier inside the 16 pivots; P = X^T X with its triangular inverse X takes half
// the time, but at order 129 and a condition of 1e5 the error was 3.3e-2 then, below 9e-3 with this); then all four wavefronts
// form W = V P and the rank-16 update of the other blocks on the MFMA units and write the new panel.
// On exit S holds the swept block (-inverse).  Pb: [16][17], Wb: [64][17] scratch.
// Returns 0 or the 1-based index (within the block) of the first non-positive pivot (valid in wave 0).
constexpr int SW_PITCH = 68;

__device__ __forceinline__ int sweep64_blocked(float *S, float *Pb, float *Wb, int tid)
{
    const int lane = tid & 63, w = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    int fail = 0;
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int c0 = kb * 16;
        if (w == 0) {
            // ---- the 16 x 16 pivot block, in registers ----
            float d[4];
            {
                const floatx4 v = *reinterpret_cast<const floatx4 *>(S + (c0 + lr) * SW_PITCH + c0 + 4 * lk);
                d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
            }
            sweep16_pivot<0>(d, lr, lk, c0, fail);
            sweep16_pivot<1>(d, lr, lk, c0, fail);
            sweep16_pivot<2>(d, lr, lk, c0, fail);
            sweep16_pivot<3>(d, lr, lk, c0, fail);
            sweep16_pivot<4>(d, lr, lk, c0, fail);
            sweep16_pivot<5>(d, lr, lk, c0, fail);
            sweep16_pivot<6>(d, lr, lk, c0, fail);
            sweep16_pivot<7>(d, lr, lk, c0, fail);
            sweep16_pivot<8>(d, lr, lk, c0, fail);
            sweep16_pivot<9>(d, lr, lk, c0, fail);
            sweep16_pivot<10>(d, lr, lk, c0, fail);
            sweep16_pivot<11>(d, lr, lk, c0, fail);
            sweep16_pivot<12>(d, lr, lk, c0, fail);
            sweep16_pivot<13>(d, lr, lk, c0, fail);
            sweep16_pivot<14>(d, lr, lk, c0, fail);
            sweep16_pivot<15>(d, lr, lk, c0, fail);
            // P = -swept block
#pragma unroll
            for (int m = 0; m < 4; ++m) Pb[lr * 17 + 4 * lk + m] = -d[m];
        }
        __syncthreads();
        // ---- rows 16w .. 16w + 15, a wavefront's own: W = V P, then S_ij -= W_i V_j^T for the three blocks outside the pivot row
        // and column, their chains side by side ----
        floatx4 wt = {0.f, 0.f, 0.f, 0.f};
        if (w != kb) {
            float b[3][4], old[3][4];
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4)
                wt = __builtin_amdgcn_mfma_f32_16x16x4f32(S[(16 * w + lr) * SW_PITCH + c0 + 4 * s4 + lk], Pb[(4 * s4 + lk) * 17 + lr], wt, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int bj = r + (r >= kb ? 1 : 0);
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) b[r][s4] = S[(16 * bj + lr) * SW_PITCH + c0 + 4 * s4 + lk];
#pragma unroll
                for (int v = 0; v < 4; ++v) old[r][v] = S[(16 * w + 4 * lk + v) * SW_PITCH + 16 * bj + lr];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) Wb[(16 * w + 4 * lk + v) * 17 + lr] = wt[v];
            floatx4 acc[3];
#pragma unroll
            for (int r = 0; r < 3; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const float x = Wb[(16 * w + lr) * 17 + 4 * s4 + lk];
#pragma unroll
                for (int r = 0; r < 3; ++r) acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[r][s4], acc[r], 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int v = 0; v < 4; ++v) S[(16 * w + 4 * lk + v) * SW_PITCH + 16 * (r + (r >= kb ? 1 : 0)) + lr] = old[r][v] - acc[r][v];
        }
        __syncthreads();
        // ---- new panel (both triangles) and pivot block ----
        if (w != kb) {
#pragma unroll
            for (int v = 0; v < 4; ++v) S[(16 * w + 4 * lk + v) * SW_PITCH + c0 + lr] = wt[v];
            *reinterpret_cast<floatx4 *>(S + (c0 + lr) * SW_PITCH + 16 * w + 4 * lk) = wt;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) S[(c0 + 4 * lk + v) * SW_PITCH + c0 + lr] = -Pb[(4 * lk + v) * 17 + lr];
        }
        __syncthreads();
    }
    return fail;
}

// The condition test of a pivot block (largest absolute row sums of the block and of its inverse) rides on the loops
// that load the block and store its inverse: in those loops thread t visits column t mod 64 in the rows t / 64 + 4 k,
// so it sums the absolute values it sees (both matrices are symmetric: column sums are row sums), leaves its part
// in nrm[(t / 64) * 64 + column], and after the next barrier one wavefront folds the four parts of every column and
// takes the largest.  nrm: 4 * 64 + 2 floats of LDS; the result goes to nrm[256 + slot], read after a later barrier.
__device__ __forceinline__ void norm_fold(float *nrm, int slot, int lane)
{
    float a = nrm[lane] + nrm[64 + lane] + nrm[128 + lane] + nrm[192 + lane];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
    if (lane == 0) nrm[256 + slot] = a;
}

// Workgroup 0 of a matrix inverts the first pivot block; workgroup r >= 1 copies block r of the first
// column panel K-major into V[0] (transposed through LDS), so that step 0 stages its panels like any
// other step.
// N > 0: the descriptors come with the launch.
template <int N>
__global__ __launch_bounds__(256) void fsweep_pivot0_kernel(const InvSeq q, const InvInline<N> own)
{
    __shared__ __attribute__((aligned(16))) float sbuf[64 * SW_PITCH];
    __shared__ __attribute__((aligned(16))) float pw[16 * 17 + 64 * 17];
    __shared__ float nrm[4 * 64 + 2];
    float (*tile)[65] = reinterpret_cast<float (*)[65]>(sbuf);
    int prob, local;
    if (!seq_locate(q, blockIdx.x, prob, local)) return;
    const int tid = threadIdx.x;
    if (N > 0 && local == 0 && tid < (int)(sizeof(InvProbF) / 4))
        reinterpret_cast<unsigned *>(const_cast<InvProbF *>(q.tab) + prob)[tid] = reinterpret_cast<const unsigned *>(&own.p[prob])[tid];
    const InvProbG pr = N > 0 ? load_prob(own.p[prob]) : load_prob(q.tab[prob]);
    if (local > 0) {
        const int g0 = local * FNB;
#pragma unroll
        for (int e = tid; e < FNB * FNB; e += 256) {
            const int c = e >> 6, k = e & 63;
            tile[c][k] = (g0 + c < pr.n) ? pr.M[(long)(g0 + c) * pr.ldm + k] : 0.f;
        }
        __syncthreads();
        for (int e = tid; e < FNB * FNB; e += 256) {
            const int k = e >> 6, c = e & 63;
            if (g0 + c < pr.n) pr.Vt[(long)k * pr.ldv + g0 + c] = tile[c][k];
        }
        return;
    }
    const int bs = min(FNB, pr.n);
    const long ldm = pr.ldm, ldw = pr.ldw;
    const float damping = pr.dptr ? *pr.dptr : pr.damping;
    const bool test = q.refine_cond >= 0.f;
    float colsum = 0.f;
    const float edge = pr.border ? pr.M[64 * ldm + (tid & 63)] : 0.f, corner = pr.border ? pr.M[64 * ldm + 64] : 0.f;     // the row behind the block
    {
        // all loads ahead of the first store (S may be any memory: one iteration would wait for the other)
        float x[FNB * FNB / 256];
#pragma unroll
        for (int u = 0; u < FNB * FNB / 256; ++u) {
            const int i = (tid >> 6) + 4 * u, j = tid & 63;
            x[u] = pr.M[min(max(i, j), bs - 1) * ldm + min(min(i, j), bs - 1)];
        }
#pragma unroll
        for (int u = 0; u < FNB * FNB / 256; ++u) {
            const int i = (tid >> 6) + 4 * u, j = tid & 63;
            const bool in = i < bs && j < bs;
            const float v = in ? x[u] + (i == j ? damping : 0.f) : (i == j ? 1.f : 0.f);
            colsum += in ? fabsf(v) : 0.f;
            sbuf[i * SW_PITCH + j] = v;
            if (test) pr.S[i * FNB + j] = in ? v : 0.f;
        }
    }
    nrm[tid] = colsum;
    __syncthreads();
    if (test && (tid >> 6) == 1) norm_fold(nrm, 0, tid & 63);       // beside the first in-register sweep of wavefront 0
    const int fail = sweep64_blocked(sbuf, pw, pw + 16 * 17, tid);   // valid in wavefront 0
    const bool whole = pr.nblk == 1;   // the block is the matrix: store the result itself, both triangles
    const bool border = whole && pr.border;
    colsum = 0.f;
    {
        float x[FNB * FNB / 256];
#pragma unroll
        for (int u = 0; u < FNB * FNB / 256; ++u) {
            const int i = (tid >> 6) + 4 * u, j = tid & 63;
            x[u] = sbuf[i * SW_PITCH + j];
            colsum += i < bs && j < bs ? fabsf(x[u]) : 0.f;
        }
        if (!border) {
#pragma unroll
            for (int u = 0; u < FNB * FNB / 256; ++u) {
                const int i = (tid >> 6) + 4 * u, j = tid & 63;
                const bool in = i < bs && j < bs;
                if (whole) {
                    // row i from the lower triangle, which is stored as both
                    if (in) pr.W[i * ldw + j] = -(j <= i ? x[u] : sbuf[j * SW_PITCH + i]);
                } else {
                    pr.P[i * FNB + j] = in ? -x[u] : 0.f;
                    if (in && j <= i) pr.W[i * ldw + j] = x[u];
                }
            }
        }
    }
    if (border) {
        // The last row and column by bordering, as the kernels of larger orders do it (invert.hip has the formulas):
        // thread (i, part) sums a quarter of row i.  y, r, z, b in pw.
        float *yv = pw, *rv = pw + 64, *zv = pw + 128, *bv = pw + 192, *red = pw + 256;
        const int i = tid & 63, part = tid >> 6;
        __syncthreads();                                     // the sweep has been read, pw is free
        if (tid < 64) bv[i] = edge;
        nrm[tid] = colsum;
        __syncthreads();
        if (part == 1 && test) norm_fold(nrm, 1, i);
        __syncthreads();
        const bool fix = test && (pr.border == 2 || nrm[256] * nrm[257] > q.refine_cond);
        auto matvec = [&](float *out, const float *in, auto row) {      // out = row(i, .) in
            float a = 0.f;
#pragma unroll
            for (int k = 0; k < 16; ++k) a = __builtin_fmaf(row(16 * part + k), in[16 * part + k], a);
            red[tid] = a;
            __syncthreads();
            if (tid < 64) out[i] = (red[i] + red[64 + i]) + (red[128 + i] + red[192 + i]);
            __syncthreads();
        };
        auto x_row = [&](int j) { return -sbuf[i * SW_PITCH + j]; };
        matvec(yv, bv, x_row);
        if (fix) {
            matvec(rv, yv, [&](int j) { return (float)pr.M[max(i, j) * ldm + min(i, j)]; });
            if (tid < 64) rv[i] = bv[i] - (rv[i] + damping * yv[i]);
            __syncthreads();
            matvec(zv, rv, x_row);
        }
        if (tid < 64) {
            float term = bv[i];
            if (fix) term += rv[i];
            red[i] = term * yv[i];
        }
        __syncthreads();
        if (tid < 64) {
            float x = red[tid];
#pragma unroll
            for (int h = 32; h > 0; h >>= 1) x += __shfl_down(x, h);
            if (tid == 0) red[0] = x;
        }
        __syncthreads();
        const float sp = corner + damping - red[0];
        const float is = 1.0f / sp;
        if (tid < 64) {
            if (fix) yv[i] += zv[i];
            const float e = -yv[i] * is;
            pr.W[64 * ldw + i] = e;
            pr.W[i * ldw + 64] = e;
        }
        __syncthreads();
        float x[FNB * FNB / 256];
#pragma unroll
        for (int u = 0; u < FNB * FNB / 256; ++u) {
            const int a = (tid >> 6) + 4 * u, b = tid & 63, hi = max(a, b), lo = min(a, b);
            x[u] = -sbuf[hi * SW_PITCH + lo] + (yv[hi] * yv[lo]) * is;
        }
#pragma unroll
        for (int u = 0; u < FNB * FNB / 256; ++u) pr.W[((tid >> 6) + 4 * u) * ldw + (tid & 63)] = x[u];
        if (tid == 0) {
            pr.W[64 * ldw + 64] = is;
            *pr.info = fail != 0 ? fail : (sp > 0.f ? 0 : 65);
        }
        return;
    }
    if (tid == 0) *pr.info = (fail <= bs) ? fail : 0;
    if (!test || whole) return;
    nrm[tid] = colsum;
    __syncthreads();
    if ((tid >> 6) == 0) {
        norm_fold(nrm, 1, tid);
        if (tid == 0) {
            // (a failed inversion leaves a NaN here: the comparison is false and the block is left alone)
            const int open = nrm[256] * nrm[257] > q.refine_cond ? 1 : 0;
            pr.gate[0] = open;
            pr.gate[2] = open;
        }
    }
}

// One step of the sweep for every tile of every active matrix (see the header of this file).
//
// Per tile and wavefront 128 fp32 MFMAs (4096 cycles of its SIMD) against the memory instructions, which cost the
// address unit that the four SIMDs share about 16 cycles each whatever their width.  So lanes move 16 bytes: the
// contraction index of MFMA step s and lane group lk is fold_k(s, lk) = 16 (s / 4) + 4 lk + s mod 4 on both operands,
// with which the values of P that a lane needs are four neighbours of a row (P is symmetric), and the second product
// has its operands swapped, so that a lane's four accumulators are neighbours of a row of the matrix.  24 memory
// instructions per wavefront and tile instead of 72; the pitch of 68 keeps both LDS operand reads (rows 4 apart)
// free of conflicts and makes room for four workgroups per CU.
// All steps of the matrices up to order 1280 of a DenseNet-201-shaped network 9.2 -> 7.1 ms of kernel time (6.0 with
// the loads of the diagonal and edge tiles as they are below), of 24
// transformer blocks of width 1024 (144 matrices of order 1024 and pivot blocks beside other kernels) 20.8 -> 11.9 ms.
__device__ __forceinline__ int fold_k(int s4, int lk) { return 16 * (s4 >> 2) + 4 * lk + (s4 & 3); }

__global__ __launch_bounds__(256, 4) void fsweep_step_kernel(const InvSeq q)
{
    typedef Tile<2, 2> T;
    constexpr int PITCH = SW_PITCH;
    // two operand buffers (the pivot-block sweep reuses them).  P is not staged: every lane keeps its 32 operand
    // values of P in registers.
    __shared__ __attribute__((aligned(16))) float Va[FNB * PITCH];   // V of the tile's row block (or the panel block)
    __shared__ __attribute__((aligned(16))) float Vb[FNB * PITCH];   // V of the tile's column block, or W^T
    __shared__ float nrm[4 * 64 + 2];                                // the condition test of the next pivot block

    int prob, t;
    if (!seq_locate(q, blockIdx.x, prob, t)) return;
    const InvProbG pr = load_prob(q.tab[prob]);
    const int K = q.step, K1 = K + 1;
    const int nblk = pr.nblk;
    if (K >= nblk) return;
    int bi, bj;
    tri_decode(t, bi, bj);
    if (K1 < nblk) {   // the next pivot tile takes block 0 and gives tile (0, 0) its own slot
        const int tp = K1 * (K1 + 1) / 2 + K1;
        if (t == 0) { bi = K1; bj = K1; }
        else if (t == tp) { bi = 0; bj = 0; }
    }
    const int tid = threadIdx.x;
    const int n = pr.n, ldv = pr.ldv;
    const long ldm = pr.ldm, ldw = pr.ldw;
    const bool first = (K == 0), last = (K1 == nblk);
    const float damping = (first && pr.dptr) ? *pr.dptr : pr.damping;
    if (bi == K && bj == K) {
        // the pivot block itself was finished by the previous launch; on the last step it still has to
        // be negated and mirrored like everything else
        if (last) {
            const int p0 = K * FNB, bs = n - p0;
            for (int e = tid; e < FNB * FNB; e += 256) {
                const int i = e >> 6, j = e & 63;
                if (i < bs && j <= i) {
                    const float v = -pr.W[(long)(p0 + i) * ldw + p0 + j];
                    pr.W[(long)(p0 + i) * ldw + p0 + j] = v;
                    pr.W[(long)(p0 + j) * ldw + p0 + i] = v;
                }
            }
        }
        return;
    }

    const int p0 = K * FNB, p1 = K1 * FNB;
    const int bs = min(FNB, n - p0);
    const int bs1 = min(FNB, n - p1);              // <= 0 when there is no next block
    const gfloat *Pk = pr.P + (K & 1) * FNB * FNB;
    const gfloat *Vk = pr.Vt + (long)(K & 1) * FNB * ldv;
    gfloat *Pn = pr.P + (K1 & 1) * FNB * FNB;
    gfloat *Sn = pr.S + (K1 & 1) * FNB * FNB;
    const gfloat *Sk = pr.S + (K & 1) * FNB * FNB;
    const bool refine = q.refine_cond >= 0.f && pr.gate[K & 1] != 0;      // uniform over the workgroup
    gfloat *Vn = pr.Vt + (long)(K1 & 1) * FNB * ldv;
    const bool panel = (bi == K) != (bj == K);
    const int ra = panel ? (bi == K ? bj : bi) : bi;   // block whose V goes to Va
    const int rb = bj;

    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 15, lk = lane >> 4;
    const bool diag = (bi == bj);
    // V of the row block and of the column block (unconditional loads, from clamped addresses), P, the tile's current
    // values (needed last): all in flight together
    const bool two = !panel && !diag;
    floatx4 sta[4], stb[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = (tid >> 4) + 16 * e, c4 = (tid & 15) * 4;
        const long row = (long)(k < bs ? k : 0) * ldv;
        const int ga = ra * FNB + c4, gb = rb * FNB + c4;
        sta[e] = *(const gfloatx4 *)(Vk + row + (ga < ldv ? ga : 0));
        stb[e] = *(const gfloatx4 *)(Vk + row + (two && gb < ldv ? gb : 0));
    }
    // ---- P operand values of this lane: P[m = (wm*2 + t)*16 + lr][k = fold_k(s, lk)] ----
    floatx4 pa[FNB / 16][T::WT];
#pragma unroll
    for (int s = 0; s < FNB / 16; ++s)
#pragma unroll
        for (int t2 = 0; t2 < T::WT; ++t2)
            pa[s][t2] = *(const gfloatx4 *)(Pk + ((wm * T::WT + t2) * 16 + lr) * FNB + 16 * s + 4 * lk);
    // oldc[ti][tj][v]: row (wm*2 + ti)*16 + lr, column (wn*2 + tj)*16 + 4*lk + v of the tile.  Of a tile that the edge of
    // the matrix cuts off, from addresses clamped into its lower triangle; what does not exist (or lies above the
    // diagonal) is left out where the values are used, and the damping is added there.  No load waits for another one:
    // under a condition each, with the damping added as they came, they cost the workgroup that goes on to the next
    // pivot block 3 us per step (orders 301 and 200: 130 -> 118 us, 1025 and 512: 484 -> 443 us).
    const bool whole = !diag && (bi + 1) * FNB <= n;      // (bj < bi: its columns exist too)
    floatx4 oldc[T::WT][T::WT];
    if (!panel) {
        const gfloat *from = first ? pr.M : pr.W;
        const long ldf = first ? ldm : ldw;
        if ((bi + 1) * FNB <= n) {
#pragma unroll
            for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
                for (int tj = 0; tj < T::WT; ++tj) {
                    const int ga = bi * FNB + (wm * T::WT + ti) * 16 + lr, gb = bj * FNB + (wn * T::WT + tj) * 16 + 4 * lk;
                    oldc[ti][tj] = *(const gufloatx4 *)(from + (long)ga * ldf + gb);
                }
        } else {
#pragma unroll
            for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
                for (int tj = 0; tj < T::WT; ++tj)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int ga = min(bi * FNB + (wm * T::WT + ti) * 16 + lr, n - 1);
                        const int gb = min(bj * FNB + (wn * T::WT + tj) * 16 + 4 * lk + v, ga);
                        oldc[ti][tj][v] = from[(long)ga * ldf + gb];
                    }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = (tid >> 4) + 16 * e, c4 = (tid & 15) * 4;
        const int na = k < bs ? n - ra * FNB - c4 : 0, nb = k < bs ? n - rb * FNB - c4 : 0;   // elements that exist
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sta[e][i] = i < na ? sta[e][i] : 0.f;
            stb[e][i] = i < nb ? stb[e][i] : 0.f;
        }
        *reinterpret_cast<floatx4 *>(Va + k * PITCH + c4) = sta[e];
        if (two) *reinterpret_cast<floatx4 *>(Vb + k * PITCH + c4) = stb[e];
    }
    __syncthreads();

    floatx4 acc[T::WT][T::WT];
#pragma unroll
    for (int a = 0; a < T::WT; ++a)
#pragma unroll
        for (int b = 0; b < T::WT; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    // acc = W^T[m][c] = sum_k P[k][m] V_a[k][c]   (P symmetric)
#pragma unroll
    for (int s4 = 0; s4 < FNB / 4; ++s4) {
        float b[T::WT];
#pragma unroll
        for (int t2 = 0; t2 < T::WT; ++t2) b[t2] = Va[fold_k(s4, lk) * PITCH + (wn * T::WT + t2) * 16 + lr];
#pragma unroll
        for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
            for (int tj = 0; tj < T::WT; ++tj)
                acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[s4 >> 2][ti][s4 & 3], b[tj], acc[ti][tj], 0, 0, 0);
    }

    if (refine) {
        // One step of iterative refinement of W = V P for an ill-conditioned pivot block S (see the blocked sweep in
        // invert.hip for the reason): R^T = V^T - S W^T, W^T += P R^T, two more 64 x 64 x 64 products.  W^T and R^T
        // pass through the LDS buffer this kind of tile does not need at this point.
        float vt[T::WT][T::WT][4];      // V^T in the layout of the accumulators
#pragma unroll
        for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
            for (int tj = 0; tj < T::WT; ++tj)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    vt[ti][tj][v] = Va[((wm * T::WT + ti) * 16 + 4 * lk + v) * PITCH + (wn * T::WT + tj) * 16 + lr];
        float *X = (panel || diag) ? Vb : Va;
        __syncthreads();   // every wave is done reading V_a
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
                for (int tj = 0; tj < T::WT; ++tj)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        X[((wm * T::WT + ti) * 16 + 4 * lk + v) * PITCH + (wn * T::WT + tj) * 16 + lr] =
                            pass == 0 ? acc[ti][tj][v] : vt[ti][tj][v];
            __syncthreads();
            floatx4 r2[T::WT][T::WT];
#pragma unroll
            for (int a = 0; a < T::WT; ++a)
#pragma unroll
                for (int b = 0; b < T::WT; ++b) r2[a][b] = pass == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[a][b];
#pragma unroll
            for (int s4 = 0; s4 < FNB / 4; ++s4) {
                float b[T::WT], sop[T::WT];     // the operand values of S are read as they are used: this path is rare
#pragma unroll
                for (int t2 = 0; t2 < T::WT; ++t2) {
                    b[t2] = X[fold_k(s4, lk) * PITCH + (wn * T::WT + t2) * 16 + lr];
                    sop[t2] = pass == 0 ? Sk[fold_k(s4, lk) * FNB + (wm * T::WT + t2) * 16 + lr] : 0.f;
                }
#pragma unroll
                for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
                    for (int tj = 0; tj < T::WT; ++tj)
                        r2[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(pass == 0 ? sop[ti] : pa[s4 >> 2][ti][s4 & 3], b[tj],
                                                                          r2[ti][tj], 0, 0, 0);
            }
            __syncthreads();   // every wave is done reading X
            if (pass == 0) {
                // R^T = V^T - S W^T takes the place of V^T
#pragma unroll
                for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
                    for (int tj = 0; tj < T::WT; ++tj)
#pragma unroll
                        for (int v = 0; v < 4; ++v) vt[ti][tj][v] -= r2[ti][tj][v];
            } else {
#pragma unroll
                for (int a = 0; a < T::WT; ++a)
#pragma unroll
                    for (int b = 0; b < T::WT; ++b) acc[a][b] = r2[a][b];
            }
        }
        // off-diagonal tiles: V_a now holds R^T, which nothing reads again (W^T goes there next)
    }

    if (panel) {
        // new panel values in place; tile (K+1, K) also feeds the next step's V'
        const bool below = ra > K;
        const bool next = (ra == K1);
#pragma unroll
        for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
            for (int tj = 0; tj < T::WT; ++tj) {
                const int c = (wn * T::WT + tj) * 16 + lr;
                const int gc = ra * FNB + c;
                const int m0 = (wm * T::WT + ti) * 16 + 4 * lk;
                if (below) {      // the pivot block has all its 64 rows: others follow it
                    if (gc < n) *(gufloatx4 *)(pr.W + (long)gc * ldw + p0 + m0) = acc[ti][tj];
                    // V'[kk = c][column p0 + m] = M[p1 + c][p0 + m]; rows kk >= bs1 are zero
                    if (next) {
                        floatx4 w = acc[ti][tj];
                        if (gc >= n) w = floatx4{0.f, 0.f, 0.f, 0.f};
                        *(gfloatx4 *)(Vn + (long)c * ldv + p0 + m0) = w;
                    }
                    continue;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = m0 + v;
                    const float w = acc[ti][tj][v];
                    if (gc < n && m < bs) {
                        if (!last) pr.W[(long)(p0 + m) * ldw + gc] = w;
                        else {   // last step: the row panel is final
                            pr.W[(long)(p0 + m) * ldw + gc] = -w;
                            pr.W[(long)gc * ldw + p0 + m] = -w;
                        }
                    }
                }
            }
        return;
    }

    // ---- W^T to LDS, then C = M_ij - W_i V_j^T ----
    // off-diagonal tiles: V_a is dead after the first product and takes W^T; diagonal tiles still need
    // V_a as V_j and put W^T into the unused second buffer
    float *Ws = diag ? Vb : Va;
    const float *Vj = diag ? Va : Vb;
    __syncthreads();   // every wave is done reading V_a
#pragma unroll
    for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
        for (int tj = 0; tj < T::WT; ++tj) {
            const int c = (wn * T::WT + tj) * 16 + lr;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = (wm * T::WT + ti) * 16 + 4 * lk + v;
                Ws[m * PITCH + c] = acc[ti][tj][v];
            }
        }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < T::WT; ++a)
#pragma unroll
        for (int b = 0; b < T::WT; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < FNB / 4; ++s4) {
        float a[T::WT], b[T::WT];
#pragma unroll
        for (int t2 = 0; t2 < T::WT; ++t2) {
            a[t2] = Ws[fold_k(s4, lk) * PITCH + (wm * T::WT + t2) * 16 + lr];
            b[t2] = Vj[fold_k(s4, lk) * PITCH + (wn * T::WT + t2) * 16 + lr];
        }
#pragma unroll
        for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
            for (int tj = 0; tj < T::WT; ++tj)
                acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[tj], a[ti], acc[ti][tj], 0, 0, 0);
    }

    // acc[ti][tj][v] = (W_i V_j^T)[a][b], a = (wm*2+ti)*16 + lr, b = (wn*2+tj)*16 + 4*lk + v
    const bool next_col = (bj == K1 && bi > K1);    // column panel of the next pivot: V'[b][ga]
    const bool next_row = (bi == K1 && bj < K1);    // row panel of the next pivot: V'[a][gb]
    const bool next_piv = (bi == K1 && bj == K1);
    if (whole) {     // not on the diagonal: never the next pivot
#pragma unroll
        for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
            for (int tj = 0; tj < T::WT; ++tj) {
                const int a = (wm * T::WT + ti) * 16 + lr, b = (wn * T::WT + tj) * 16 + 4 * lk;
                const int ga = bi * FNB + a, gb = bj * FNB + b;
                floatx4 c;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    c[v] = oldc[ti][tj][v] - acc[ti][tj][v];
                    if (next_col) Vn[(long)(b + v) * ldv + ga] = c[v];
                    if (last) {
                        c[v] = -c[v];
                        pr.W[(long)(gb + v) * ldw + ga] = c[v];
                    }
                }
                if (next_row) *(gfloatx4 *)(Vn + (long)a * ldv + gb) = c;
                *(gufloatx4 *)(pr.W + (long)ga * ldw + gb) = c;
            }
        return;
    }
    __syncthreads();   // Va is reused below when this tile is the next pivot
#pragma unroll
    for (int ti = 0; ti < T::WT; ++ti)
#pragma unroll
        for (int tj = 0; tj < T::WT; ++tj) {
            const int a = (wm * T::WT + ti) * 16 + lr;
            const int ga = bi * FNB + a;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = (wn * T::WT + tj) * 16 + 4 * lk + v;
                const int gb = bj * FNB + b;
                const bool ok = (ga < n && gb < n && (!diag || gb <= ga));
                float c = 0.f;
                if (ok) {
                    c = (oldc[ti][tj][v] + (first && ga == gb ? damping : 0.f)) - acc[ti][tj][v];
                    if (last) {
                        pr.W[(long)ga * ldw + gb] = -c;
                        pr.W[(long)gb * ldw + ga] = -c;
                    } else if (!next_piv) {
                        pr.W[(long)ga * ldw + gb] = c;
                    }
                }
                if (next_col && ga < n) Vn[(long)b * ldv + ga] = ok ? c : 0.f;
                if (next_row && gb < n) Vn[(long)a * ldv + gb] = ok ? c : 0.f;
                if (next_piv) Va[a * PITCH + b] = c;
            }
        }
    if (!next_piv) return;

    // ---- this workgroup holds the next pivot block: invert it now ----
    __syncthreads();
    {
        const bool test = q.refine_cond >= 0.f;
        float colsum = 0.f;
        for (int e = tid; e < FNB * FNB; e += 256) {
            const int i = e >> 6, j = e & 63;
            float v = (i == j) ? 1.f : 0.f;
            const bool in = i < bs1 && j < bs1;
            if (in) {
                v = (j <= i) ? Va[i * PITCH + j] : Va[j * PITCH + i];
                colsum += fabsf(v);
            }
            Vb[i * SW_PITCH + j] = v;
            if (test) Sn[i * FNB + j] = in ? v : 0.f;
        }
        nrm[tid] = colsum;
        __syncthreads();
        if (test && (tid >> 6) == 1) norm_fold(nrm, 0, tid & 63);   // beside the first in-register sweep of wavefront 0
        const int fail = sweep64_blocked(Vb, Va, Va + 16 * 17, tid);
        colsum = 0.f;
        for (int e = tid; e < FNB * FNB; e += 256) {
            const int i = e >> 6, j = e & 63;
            const bool in = (i < bs1 && j < bs1);
            const float v = Vb[i * SW_PITCH + j];
            if (in) colsum += fabsf(v);
            Pn[i * FNB + j] = in ? -v : 0.f;
            if (in && j <= i) pr.W[(long)(p1 + i) * ldw + p1 + j] = v;
        }
        // launches of one sequence are ordered, so the first failing pivot wins
        if (fail != 0 && fail <= bs1 && tid == 0 && *pr.info == 0) *pr.info = p1 + fail;
        if (!test) return;
        nrm[tid] = colsum;
        __syncthreads();
        if ((tid >> 6) == 0) {
            norm_fold(nrm, 1, tid);
            if (tid == 0) {
                const int open = nrm[256] * nrm[257] > q.refine_cond ? 1 : 0;
                pr.gate[K1 & 1] = open;
                if (open) pr.gate[2] = 1;
            }
        }
    }
}

}  // namespace kfac
