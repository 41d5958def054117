// C = A^T B for fp32 operands (both K-major) on the bf16 MFMA units, at fp32 accuracy: the split-bf16 core of
// split_common.hpp with the epilogues of the preconditioning (Eq. 5 of the DP-KFAC paper) and of the blocked
// inversion's rank-k updates and panel products (section 5.2).
//
// Bound: bf16 MFMA, six products per fp32 product (2.5 PFLOP/s / 6 = 417 TFLOP/s in flops of the definition;
// v_mfma_f32_32x32x16_bf16 reaches 2.1 of the 2.5 when fed from registers).  Two workgroups share a CU, so the
// prologue and the read-modify-write epilogue of one run beside the MFMAs of the other.
#pragma once

#include "split_common.hpp"

namespace kfac {

struct GemmSProb {
    const float *A;
    const float *B;
    float *C;
    int lda, ldb, ldc;
    int M, N, K;
    int tI, tJ;      // tiles over M (256 rows) and N (128 columns)
    int blk_start;
    int mode;        // kStore, kSubLowerSkip, kSubRect or kAddRect
    int p0, p1;
    int doff;        // the subtracting modes touch n <= m + doff (0 for kSubLowerSkip)
    const int *gate; // null, or two float bit patterns: leave C alone unless their product exceeds gate_cond
    float gate_cond;
    int tiles;       // of one K slice
    int kper;        // rows of K per slice (a multiple of 16, or K); slice i stores into C + i cstride
    long cstride;
    int abytes;      // bytes from A to the end of its buffer: what lies past it reads as zero
};

constexpr int kMaxGemmS = 96;        // products per launch (a 10 KB kernel argument)

struct GemmSTable {
    int count;
    int xcd[9];      // XCD x takes the tiles xcd[x] .. xcd[x + 1] - 1
    int starts[kMaxGemmS];
    GemmSProb p[kMaxGemmS];
};

// column tiles of tile row i: all of them, or those that reach the line n = m + doff
__host__ __device__ inline int split_row_len(int mode, int tJ, int doff, int i)
{
    if (mode == kStore) return tJ;
    const long last = ((long)i * S_BM + S_BM - 1 + doff) / S_BN + 1;
    return (int)(last < tJ ? last : tJ);
}

__global__ __launch_bounds__(256, 2) void gemm_split_kernel(const GemmSTable tab)
{
    __shared__ __attribute__((aligned(16))) SplitLds L;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = w & 1;

    // Every XCD (workgroup i runs on XCD i mod 8) takes a contiguous range of tile numbers, so that its L2 sees few
    // operand panels; the ranges are of equal K stages, not of equal tiles (with equal tiles the XCDs that got the
    // deep products of a mixed launch worked twice as long as the others).  The tiles of a product are numbered in
    // groups of four tile rows, column by column inside a group: the tiles that run at the same time share their A
    // panels (four per group) and their B panels (one per four tiles).
    const int x = blockIdx.x & 7;
    const int bid = tab.xcd[x] + (int)(blockIdx.x >> 3);
    if (bid >= tab.xcd[x + 1]) return;
    int pi = 0, hi = tab.count - 1;
    while (pi < hi) {
        const int mid = (pi + hi + 1) >> 1;
        if (bid >= tab.starts[mid]) pi = mid;
        else hi = mid - 1;
    }
    const GemmSProb &pr = tab.p[pi];
    // uniform over the workgroup, before any barrier or load
    if (pr.gate && !(__int_as_float(pr.gate[0]) * __int_as_float(pr.gate[1]) > pr.gate_cond)) return;
    int local = bid - pr.blk_start;
    const int slice = local / pr.tiles, k0 = slice * pr.kper, K = min(pr.kper, pr.K - k0);
    local -= slice * pr.tiles;
    int I, J;
    const bool lower = pr.mode != kStore;         // read-modify-write below the line n = m + doff
    const bool rows_skip = pr.mode == kSubLowerSkip;
    const bool add = pr.mode == kAddRect;
    {
        auto row_len = [&](int i) { return i >= pr.tI ? 0 : split_row_len(pr.mode, pr.tJ, pr.doff, i); };
        int g = 0;
        for (;;) {
            const int c = row_len(4 * g) + row_len(4 * g + 1) + row_len(4 * g + 2) + row_len(4 * g + 3);
            if (local < c) break;
            local -= c;
            ++g;
        }
        // inside the group: column J holds the rows whose length exceeds J (row lengths grow with i)
        const int l0 = row_len(4 * g), l1 = row_len(4 * g + 1), l2 = row_len(4 * g + 2), l3 = row_len(4 * g + 3);
        J = 0;
        for (;;) {
            const int c = (J < l0) + (J < l1) + (J < l2) + (J < l3);
            if (local < c) break;
            local -= c;
            ++J;
        }
        // the local-th row (in increasing order) among those with length > J
        int i = 0;
        for (int seen = 0;; ++i) {
            const int len = i == 0 ? l0 : (i == 1 ? l1 : (i == 2 ? l2 : l3));
            if (J < len) {
                if (seen == local) break;
                ++seen;
            }
        }
        I = 4 * g + i;
    }
    const int m0 = I * S_BM, n0 = J * S_BN;
    if (lower) {
        // tiles wholly inside the pivot rows or columns are left untouched
        const int m1 = min(m0 + S_BM, pr.M), n1 = min(n0 + S_BN, pr.N);
        if ((rows_skip && m0 >= pr.p0 && m1 <= pr.p1) || (n0 >= pr.p0 && n1 <= pr.p1)) return;
    }

    const long lda = pr.lda, ldb = pr.ldb;
    SplitSrc<kRows> src;
    {
        // the host checked: below 2 GiB.  (A slice past the last row has no stages.)
        const long sa = (long)min(k0, pr.K) * lda, sb = (long)min(k0, pr.K) * ldb;
        const long na = max(0l, pr.abytes - sa * 4), nb = (long)pr.K * ldb * 4 - sb * 4;
        src.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.A + sa), 0, (int)na, 0x00020000);
        src.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.B + sb), 0, (int)nb, 0x00020000);
        src.lda4 = (unsigned)lda * 4u;
        src.ldb4 = (unsigned)ldb * 4u;
        src.nstages = (max(K, 0) + S_KT - 1) / S_KT;
        src.init_thread(tid);
        src.lim_a = pr.M - m0;
        src.lim_b = pr.N - n0;
        const int ca = m0 + src.col_a(0), cb = n0 + src.col_b(0);
        src.va[0] = ca < pr.M ? (unsigned)ca * 4u + 4u * (unsigned)src.kq * src.lda4 : W_OOB;
        src.vb[0] = cb < pr.N ? (unsigned)cb * 4u + 4u * (unsigned)src.kq * src.ldb4 : W_OOB;
    }
    const int lr = lane & 31, lg = lane >> 5;
    // row tiles this wavefront has to compute: none above the line n = m + doff or past the edges
    const int mleft = pr.M - (m0 + wm * (S_BM / 2));
    const bool idle = (lower && (n0 + wn * 64 > m0 + wm * (S_BM / 2) + S_BM / 2 - 1 + pr.doff)) || mleft <= 0 ||
                      n0 + wn * 64 >= pr.N;
    const int rows = idle ? 0 : (mleft + 31) / 32;
    floatx16 acc[8];
    float none[4];
    const float unscale = split_tile<kRows, false, false>(src, L, acc, none, 0, rows, wm, wn, tid);
    if (idle) return;

    // ---- epilogue: acc[ti*2 + tj][v] = C[m0 + wm*S_BM/2 + ti*32 + 8*(v>>2) + 4*lg + (v&3)][n0 + wn*64 + tj*32 + lr]
    // A lane of the MFMA result holds single elements of many rows: written or updated from there, every memory
    // instruction moves 4 bytes per lane.  Instead each wavefront passes its part through LDS (the ring is free
    // now), 32 rows x 64 columns at a time, and reads it back with 16 lanes along a row, four columns each: the
    // accesses to C are 16 bytes per lane and 256 contiguous bytes per row.  (C need not be 16-byte aligned: buffer
    // accesses ask for 4.)
    // Loads and stores share one counter and complete in order: a load issued after a store is not seen before that
    // store has been acknowledged.  So the old values are fetched in two batches of two chunks, the results stay in
    // registers, and all stores come last.
    // What limits this code is its size: it runs once per workgroup, and every line of it that is not in the
    // instruction cache is fetched from memory while the wavefront waits.  An unrolled element-wise path for the
    // chunks that the bounds, the line n = m + doff or the pivot rows and columns cut through (100 KB of code) made the
    // epilogue take 40 us whatever K, more than half of a rank-256 update.  Such a chunk is now read like any other, and
    // stored with a 16-byte access by the lanes whose four columns are all wanted and up to three 4-byte accesses by
    // the others; what must not be written gets an offset outside the buffer.
    const int mw = m0 + wm * (S_BM / 2), nw = n0 + wn * 64;
    const int ldc = pr.ldc;
    constexpr int EP = 68;                                   // LDS row pitch of a chunk (floats)
    float *wl = reinterpret_cast<float *>(L.ring) + w * 32 * EP;
    const int rr = lane >> 4, c4 = (lane & 15) * 4;
    // the host checked that M rows of C are below 2 GiB
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(pr.C + slice * pr.cstride, 0, (int)((long)pr.M * ldc * 4), 0x00020000);
    const unsigned vo = (unsigned)(rr * ldc + c4) * 4u;
    const float sign = (lower && !add) ? -unscale : unscale;
    auto row_off = [&](int ti, int q) { return (unsigned)((mw + ti * 32 + 4 * q) * ldc + nw) * 4u; };
    floatx4 out[4][8];
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += 2) {
#pragma unroll
        for (int ti = t0; ti < t0 + 2; ++ti)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                out[ti][q] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (lower) {
                    const sint4 v = __builtin_bit_cast(sint4, __builtin_amdgcn_raw_buffer_load_b128(rc, vo + row_off(ti, q), 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[ti][q][e] = __int_as_float(v[e]);
                }
            }
#pragma unroll
        for (int ti = t0; ti < t0 + 2; ++ti) {
#pragma unroll
            for (int tj = 0; tj < 2; ++tj) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    wl[(8 * (v >> 2) + 4 * lg + (v & 3)) * EP + tj * 32 + lr] = acc[ti * 2 + tj][v];
            }
            // (LDS operations of one wavefront complete in order: no barrier between these writes and the reads)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const floatx4 val = *reinterpret_cast<const floatx4 *>(wl + (4 * q + rr) * EP + c4);
#pragma unroll
                for (int e = 0; e < 4; ++e) out[ti][q][e] = __builtin_fmaf(sign, val[e], out[ti][q][e]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // (The whole offset of an access sits in its vector register: the range check looks at that one alone; and with an
    // offset in a scalar register the compiler takes it that a wide store has read its data at once, where on this chip
    // the instruction behind it could still change the last lanes' last word, seen in the results.)
    // Columns n .. n + 3 of row m are wanted as far as wanted(m) says; p0 and p1 are multiples of 4 (or p1 is past the
    // edge), so a pivot band takes a lane's columns whole.
    const int n = nw + c4;
    const bool pcol = lower && n >= pr.p0 && n < pr.p1;
    auto wanted = [&](int m) {
        const bool skip = m >= pr.M || pcol || (rows_skip && m >= pr.p0 && m < pr.p1);
        const int limit = lower ? min(pr.N, m + pr.doff + 1) : pr.N;
        return skip ? 0 : limit - n;
    };
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int have = wanted(mw + ti * 32 + 4 * q + rr);
            const unsigned o = vo + row_off(ti, q);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(suint4, out[ti][q]), rc, have >= 4 ? o : W_OOB, 0, 0);
            if (__any(have > 0 && have < 4)) {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[ti][q][e]), rc,
                                                          have < 4 && e < have ? o + 4u * (unsigned)e : W_OOB, 0, 0);
            }
        }
}

}  // namespace kfac
