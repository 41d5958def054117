// X^T X partial products for fp32 X (row-major patch matrices and linear-layer inputs, NCHW inputs of 1x1
// convolutions and output gradients) on the bf16 MFMA units at fp32 accuracy: the split-bf16 core of
// split_common.hpp applied to the Kronecker factors of Eq. 4 of the DP-KFAC paper.
//
// A workgroup of four wavefronts owns a 256 x 128 tile of the lower triangle (256 columns of X as rows of the
// factor, 128 as columns) for one K slice.  Partial tiles go to the workspace in the 256 x 256 block layout of the
// bf16 kernel (two workgroup tiles per block), so the same reduction finishes them (fixed order, running average,
// mirror image).  The two tiles of a diagonal block take B's fragments from A's: a third less to load and convert.
//
// The bias border (column sums of X) is summed on the side, in plain fp32, by the threads of the first tile of every
// diagonal block from the values they load for A.
#pragma once

#include "split_common.hpp"
#include "syrk_types.hpp"

namespace kfac {

// workgroup tiles (256 x 128) of the lower triangle of a d x d factor
__host__ __device__ inline int syrk_split_tiles(int d)
{
    const int tI = (d + S_BM - 1) / S_BM, tJ = (d + S_BN - 1) / S_BN;
    int n = 0;
    for (int i = 0; i < tI; ++i) n += (2 * i + 2 < tJ) ? 2 * i + 2 : tJ;
    return n;
}

// MASK: some NCHW problem of the launch has a number of positions that is no multiple of 4
template <int LAYOUT, bool MASK>
__global__ __launch_bounds__(256, 2) void syrk_split_kernel(const SyrkTable tab)
{
    __shared__ __attribute__((aligned(16))) SplitLds L;
    typedef SplitSrc<LAYOUT> Src;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = w & 1;

    // every XCD takes a contiguous range of workgroups: the tiles of a K slice, which share its panels, are
    // neighbours and meet in one L2
    const int bid = xcd_block_id();
    int pi = 0, hi = tab.count - 1;
    while (pi < hi) {
        const int mid = (pi + hi + 1) >> 1;
        if (bid >= tab.starts[mid]) pi = mid;
        else hi = mid - 1;
    }
    const SyrkProb &pr = tab.p[pi];
    const int d = pr.d;
    const int tJ = (d + S_BN - 1) / S_BN;
    const int bps = syrk_split_tiles(d);
    const int local = bid - pr.blk_start;
    const int split = local / bps;
    int rest = local - split * bps;
    int I = 0;
    for (;;) {
        const int c = min(tJ, 2 * I + 2);
        if (rest < c) break;
        rest -= c;
        ++I;
    }
    const int J = rest;
    const int m0 = I * S_BM, n0 = J * S_BN;
    const bool sums = pr.has_bias && J == 2 * I;      // first tile of a diagonal block: column sums of the A panel

    // ---- K range of this slice ----
    const long t0 = (long)split * pr.tiles_per_split;
    Src src;
    src.init_thread(tid);
    src.lim_a = d - m0;
    src.lim_b = d - n0;
    if (LAYOUT == kRows) {
        const long ktiles = (pr.K + S_KT - 1) / S_KT;
        const long t1 = (t0 + pr.tiles_per_split < ktiles) ? t0 + pr.tiles_per_split : ktiles;
        const long row0 = t0 * S_KT;
        const long left = (pr.K - row0) * pr.ld * 4;
        float *base = const_cast<float *>(reinterpret_cast<const float *>(pr.x) + row0 * pr.ld);
        src.ra = __builtin_amdgcn_make_buffer_rsrc(base, 0, left > 0x7fffffffl ? 0x7fffffff : (int)left, 0x00020000);
        src.rb = src.ra;
        src.nstages = (int)(t1 - t0);
        src.lda4 = src.ldb4 = (unsigned)pr.ld * 4u;
        const int ca = m0 + src.col_a(0), cb = n0 + src.col_b(0);
        src.va[0] = ca < d ? (unsigned)ca * 4u + 4u * (unsigned)src.kq * src.lda4 : W_OOB;
        src.vb[0] = cb < d ? (unsigned)cb * 4u + 4u * (unsigned)src.kq * src.ldb4 : W_OOB;
    } else {
        src.hw = pr.hw;
        const int nimg = (int)(pr.K / pr.hw);
        src.tpi = (pr.hw + S_KT - 1) / S_KT;
        const long ktiles = (long)nimg * src.tpi;
        const long t1 = (t0 + pr.tiles_per_split < ktiles) ? t0 + pr.tiles_per_split : ktiles;
        src.nstages = (int)(t1 - t0);
        src.img0 = (int)(t0 / src.tpi);
        src.kt0 = (int)(t0 - (long)src.img0 * src.tpi);
        src.img_bytes = (unsigned)pr.ctot * (unsigned)pr.hw * 4u;
        float *base = const_cast<float *>(reinterpret_cast<const float *>(pr.x));
        // the host checked that the tensor is below 2 GiB
        src.ra = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)((long)nimg * src.img_bytes), 0x00020000);
        src.rb = src.ra;
        const unsigned q = 16u * (unsigned)src.kq;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = m0 + src.col_a(i);
            src.va[i] = c < d ? (unsigned)c * (unsigned)pr.hw * 4u + q : W_OOB;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = n0 + src.col_b(i);
            src.vb[i] = c < d ? (unsigned)c * (unsigned)pr.hw * 4u + q : W_OOB;
        }
    }

    floatx16 acc[8];
    float csum[4];
    const int lr = lane & 31, lg = lane >> 5;
    // row tiles of this wavefront's 128 x 64 part: none wholly above the diagonal or past the edges
    const int mleft = d - (m0 + wm * 128);
    const bool idle = n0 + wn * 64 > m0 + wm * 128 + 127 || mleft <= 0 || n0 + wn * 64 >= d;
    const int rows = idle ? 0 : (mleft + 31) / 32;
    const float unscale = J >= 2 * I ? split_tile<LAYOUT, true, MASK>(src, L, acc, csum, n0 - m0, rows, wm, wn, tid)
                                     : split_tile<LAYOUT, false, MASK>(src, L, acc, csum, 0, rows, wm, wn, tid);

    // ---- partial tile -> block (bi, bj) = (I, J / 2) of the slice, columns 128 (J & 1) .. of the block ----
    const int nblk = pr.nb * (pr.nb + 1) / 2;
    if (sums) {
        float *cs = pr.partial + (long)pr.splits * nblk * (S_BM * S_BM) + ((long)split * pr.nb + I) * S_BM;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float s = src.sum_quarters(csum[i]);
            if (src.kq == 0) cs[src.col_a(i)] = s;
        }
    }
    if (idle) return;
    const int blk = I * (I + 1) / 2 + (J >> 1);
    // Each wavefront passes its 128 x 64 part through LDS, 32 rows at a time, and reads it back with 16 lanes along
    // a row: the stores are 16 bytes per lane and 256 contiguous bytes per row instead of 4 bytes per lane.  (LDS
    // operations of one wavefront complete in order: no barrier between writes and reads; every wavefront is past
    // the last barrier of the K loop.)
    float *dst = pr.partial + ((long)split * nblk + blk) * (S_BM * S_BM) + (J & 1) * S_BN + wn * 64;
    constexpr int EP = 68;                                   // LDS row pitch of a chunk (floats)
    float *wl = reinterpret_cast<float *>(L.ring) + w * 32 * EP;
    const int rr = lane >> 4, c4 = (lane & 15) * 4;
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                wl[(8 * (v >> 2) + 4 * lg + (v & 3)) * EP + tj * 32 + lr] = acc[ti * 2 + tj][v];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int row = 4 * q + rr;
            const floatx4 val = *reinterpret_cast<const floatx4 *>(wl + row * EP + c4) * unscale;
            *reinterpret_cast<floatx4 *>(dst + (long)(wm * 128 + ti * 32 + row) * S_BM + c4) = val;
        }
    }
}

}  // namespace kfac
