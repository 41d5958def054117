// The split-bf16 product core shared by gemm_split.hpp and syrk_split.hpp: tiles of C = A^T B for fp32 operands on
// the bf16 MFMA units, at fp32 accuracy for every finite input.
//
// Arithmetic.  Every operand value, times 2^16, is cut into three bf16 pieces, x = x1 + x2 + x3 with x1 = bf16(x),
// x2 = bf16(x - x1) and x3 the rest, x1 and x2 rounded to nearest.  The cut is exact: x - x1 has 16 bits left,
// x - x1 - x2 seven, and bf16 has the exponents of fp32, so that nothing depends on how an operand's values compare with
// each other.  (The last bit of a bf16 number is at least 2^-133, of an fp32 number 2^-149: without the 2^16, values
// below 2^-110 lost bits of their last piece, those of 2^-120 kept 14 of 24.  The results are divided by 2^32.)
// The product keeps the six largest of the nine piece products,
//     a b  ~  a1 b1 + a1 b2 + a2 b1 + a1 b3 + a3 b1 + a2 b2,
// each exact in the fp32 accumulator of v_mfma_f32_32x32x16_bf16.  |x2| <= 2^-8 |x| and |x3| <= 2^-17 |x|, so the terms
// left out (a2 b3, a3 b2, a3 b3) are below 2^-24 |a b| and as often positive as negative.  The rounding matters: the
// MFMA cuts off the low bits of aligned addends, and with truncated pieces, which all have the sign of x, this
// adds up on operands of one sign (K = 4096, post-ReLU data: 5.3e-6 of the result with truncated pieces, 5.9e-7 with
// rounded ones, 4.9e-7 on the fp32 MFMA; zero-mean data 1.0e-6, 1.0e-6 and 1.2e-6).
// (Two fp16 pieces of a column-scaled value and three products take half the MFMAs, but hold a value to 2^-33 of the
// largest one of its column only: a feature of scale 2^24 whose inverse column is as much smaller came out with an error of
// 1e-3, and no test on the results finds every such case.)
//
// Infinities, NaN, values from 2^112 and sums from 2^96 on give accumulators that are not finite (inf - inf in the
// cut).  A tile with such a result is computed once more on the fp32 MFMA, which leaves what fp32 arithmetic gives.
//
// Pipeline.  A workgroup of four wavefronts owns a tile of 256 x 128, a wavefront 128 x 64 of it.  K goes in stages of
// 16 rows = one MFMA step.  A thread loads four k of four columns of A and of two of B, with 16- and 8-byte loads (a load
// instruction costs a wavefront about 16 cycles of the address unit whatever its width), two stages ahead.  The values
// are converted ONCE per workgroup and written to LDS as halves of ready fragments (a fragment = the eight k of one
// column and piece = 16 bytes) in two buffers (74 KB: two workgroups per CU), one barrier per stage.  The conversion
// (8.5 VALU operations per value) runs between the MFMAs, about four operations beside each of the 48 of a wavefront.
// Fragments of consecutive columns are spread over LDS by split_slot so that the MFMA reads (32 consecutive columns) and
// the writes (every fourth column) both touch every bank group equally.
// Bound: MFMA.  4096^3: the units are busy 80 % of the cycles, no bank conflicts, and the chip, short of power, runs at
// about 1.5 GHz.  624 us (1320 TFLOP/s of bf16 products) where the form without the 2^16 takes 614; 1024^3, one tile per
// CU at most, 77 against 73 us.  (On a card where that form takes 705 us: the barrier ahead of the last MFMAs of a stage,
// with the first fragments of the next one read behind it, 735 us; six products of truncated pieces cut by every wavefront
// for itself, 779 us.)
#pragma once

#include <type_traits>

#include "wave_common.hpp"

namespace kfac {

constexpr int S_BM = 256;                     // rows of C per workgroup (columns of A)
constexpr int S_BN = 128;                     // columns of C per workgroup (columns of B)
constexpr int S_KT = 16;                      // rows of the operands per stage

typedef __bf16 sbf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned suint4 __attribute__((ext_vector_type(4)));
typedef unsigned suint2 __attribute__((ext_vector_type(2)));
typedef int sint4 __attribute__((ext_vector_type(4)));
typedef int sint2 __attribute__((ext_vector_type(2)));

constexpr int kSplitShift = 16;                          // every operand value times 2^16 ...
constexpr float kSplitUnscale = 1.f / 4294967296.f;      // ... and every sum of products times 2^-32

// The cut of four values (the k of one column), in eight steps of about four operations that the K loop spreads over
// its MFMAs.  Rounded to bf16 (ties away from zero): half a unit added to the bit pattern, which may carry into the exponent.
// (v_cvt_pk_bf16_f32 issues at a quarter of the rate of these.)
struct SplitCut {
    unsigned t[4];
    float h[4];
    __device__ __forceinline__ void scale(float (&x)[4]) const
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_ldexpf(x[e], kSplitShift);
    }
    __device__ __forceinline__ void half(const float (&x)[4], int from, int to)
    {
#pragma unroll
        for (int e = from; e < to; ++e) t[e] = __float_as_uint(x[e]) + 0x8000u;
    }
    __device__ __forceinline__ void top(int from, int to)
    {
#pragma unroll
        for (int e = from; e < to; ++e) h[e] = __uint_as_float(t[e] & 0xffff0000u);
    }
    __device__ __forceinline__ void rest(float (&x)[4], int from, int to) const
    {
#pragma unroll
        for (int e = from; e < to; ++e) x[e] -= h[e];
    }
    // the upper halves of four words
    __device__ __forceinline__ suint2 pack() const
    {
        return suint2{__builtin_amdgcn_perm(t[1], t[0], 0x07060302u), __builtin_amdgcn_perm(t[3], t[2], 0x07060302u)};
    }
    __device__ __forceinline__ suint2 pack_last(const float (&x)[4]) const
    {
        return suint2{__builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u),
                      __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07060302u)};
    }
};

// Place of column c (of up to 256) among the fragments of one k group and piece: groups of 128 columns, inside them
// column 4 q + j goes to 32 j + (q ^ swizzle(j)).
__host__ __device__ constexpr int split_swz(int j) { return ((j & 1) << 3) | ((j >> 1) << 2) | ((j & 1) << 1); }
__device__ __forceinline__ int split_slot(int c)
{
    return (c & ~127) | ((c & 3) << 5) | (((c & 127) >> 2) ^ split_swz(c & 3));
}

// LDS of a workgroup: the stage buffers of fragments and a flag word
struct SplitLds {
    static constexpr int KG_A = 3 * S_BM + 1;                // fragments from k group 0 to 1 (three pieces; odd: the two
    static constexpr int KG_B = 3 * S_BN + 1;                //   halves of a wavefront read different bank groups)
    static constexpr int FRAG_B = 2 * KG_A;                  // first fragment of B
    static constexpr int BUF = 2 * KG_A + 2 * KG_B;          // fragments per stage buffer
    static constexpr int EPI = 4 * 32 * 68 / 4;              // the epilogue's chunks, in 16-byte units
    static_assert(2 * BUF >= EPI, "the epilogue reuses the ring");
    suint4 ring[2 * BUF];
    int redo;
};

// Where the operands of a tile come from, and which part of a stage a thread handles: four k (quarter kq of the
// stage) of the columns col_a(0 .. 3) of A and col_b(0 .. 1) of B.
// kRows: element (k, c) at base + k ld + c.  The columns of a thread are neighbours: one load instruction per row.
// kNCHW: element (k = n hw + p, c) at (n ctot + c) hw + p; a stage never crosses an image.  The four k are
// neighbours: one 16-byte load per column, four neighbouring lanes the 16 positions of a channel.
template <int LAYOUT>
struct SplitSrc {
    __amdgpu_buffer_rsrc_t ra, rb;
    unsigned va[LAYOUT == kRows ? 1 : 4], vb[LAYOUT == kRows ? 1 : 2];   // byte offset of the column(s), or W_OOB
    unsigned lda4, ldb4;           // kRows: row pitch in bytes
    bool down = false;             // kRows: from the last stage to the first
    int ahead = 0, back = 0;       // kRows: beginning with stage `ahead`, the ones before it come last, from place `back` on
    int lim_a, lim_b;              // columns of the tile that exist
    int nstages;
    int hw, tpi, img0, kt0, ii, ik;   // kNCHW: image walk
    unsigned img_bytes;
    int cg, kq;                    // this thread's column group (0 .. 63) and quarter of the stage

    struct Raw {
        float a[4][4], b[2][4];  // [column][k]
    };

    __device__ __forceinline__ void init_thread(int tid)
    {
        const int lane = tid & 63, w = tid >> 6;
        cg = 16 * w + (LAYOUT == kRows ? (lane >> 1) & 15 : lane >> 2);
        kq = LAYOUT == kRows ? 2 * (lane >> 5) + (lane & 1) : lane & 3;
    }
    __device__ __forceinline__ int col_a(int i) const { return LAYOUT == kRows ? 4 * cg + i : 64 * i + cg; }
    __device__ __forceinline__ int col_b(int i) const { return LAYOUT == kRows ? 2 * cg + i : 64 * i + cg; }
    // sum over the threads that hold the other k of the same columns
    static __device__ __forceinline__ float sum_quarters(float s)
    {
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, LAYOUT == kRows ? 32 : 2);
        return s;
    }

    __device__ __forceinline__ void rewind()
    {
        ii = img0;
        ik = kt0;
    }
    // Where the stage to be loaded next begins.
    struct At {
        bool live;                 // false: a stage past the end, all zeros
        unsigned sa, sb;           // byte offsets of its first row (kNCHW: sa, of its first position)
        int valid;                 // kNCHW: its positions inside the image
    };
    // kNCHW: the walk is sequential; kRows: any stage
    __device__ __forceinline__ At at(int g)
    {
        At p;
        p.live = g < nstages;
        if constexpr (LAYOUT == kRows) {
            const int row = (down ? nstages - 1 - g : g < back ? g + ahead : g - back) * S_KT;
            p.sa = p.live ? (unsigned)row * lda4 : 0u;
            p.sb = p.live ? (unsigned)row * ldb4 : 0u;
            p.valid = S_KT;
        } else {
            p.valid = min(S_KT, hw - ik * S_KT);
            p.sa = p.sb = p.live ? (unsigned)ii * img_bytes + (unsigned)(ik * S_KT * 4) : 0u;
            if (++ik == tpi) { ik = 0; ++ii; }
        }
        return p;
    }
    template <int N>
    static __device__ __forceinline__ void load_rows(float (&x)[N][4], __amdgpu_buffer_rsrc_t rsrc, unsigned vo, unsigned so,
                                                     unsigned pitch)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (N == 4) {
                const sint4 v = __builtin_bit_cast(sint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so + (unsigned)e * pitch, 0));
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i][e] = __int_as_float(v[i]);
            } else {
                const sint2 v = __builtin_bit_cast(sint2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, so + (unsigned)e * pitch, 0));
#pragma unroll
                for (int i = 0; i < 2; ++i) x[i][e] = __int_as_float(v[i]);
            }
        }
    }
    static __device__ __forceinline__ void load_pos(float (&x)[4], __amdgpu_buffer_rsrc_t rsrc, unsigned vo, unsigned so)
    {
        const sint4 v = __builtin_bit_cast(sint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __int_as_float(v[e]);
    }
    // kNCHW: a lane whose four positions all lie past the image loads nothing; partly valid groups are cut at the
    // conversion
    __device__ __forceinline__ bool in(const At &p) const { return LAYOUT == kRows ? p.live : p.live && 4 * kq < p.valid; }
    __device__ __forceinline__ void load_a(Raw &r, const At &p)
    {
        if constexpr (LAYOUT == kRows) {
            load_rows<4>(r.a, ra, in(p) ? va[0] : W_OOB, p.sa, p.live ? lda4 : 0u);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) load_pos(r.a[i], ra, in(p) ? va[i] : W_OOB, p.sa);
        }
    }
    __device__ __forceinline__ void load_b(Raw &r, const At &p)
    {
        if constexpr (LAYOUT == kRows) {
            load_rows<2>(r.b, rb, in(p) ? vb[0] : W_OOB, p.sb, p.live ? ldb4 : 0u);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) load_pos(r.b[i], rb, in(p) ? vb[i] : W_OOB, p.sb);
        }
    }
};

// The K loop of a tile.  acc: eight accumulator tiles, [ti][tj], of the wavefront's 128 x 64 part, times the inverse of
// what is returned (the same for the whole workgroup).  SHARED: B's columns
// are columns boff .. boff + 127 of A (tiles on the diagonal of X^T X; boff is 0 or 128): B is neither loaded nor
// converted, and the sums of this thread's columns of A over its k go to csum.  MASK: some NCHW problem of the launch has a
// number of positions that is no multiple of 4 (positions past the end of an image hold the next channel's data).
// `rows`: row tiles (of 32 rows) of the wavefront's part that are wanted.  0: it only helps with the staging; 1: it
// multiplies that one (the bias column makes orders of 2^n + 1 the rule here: a tile for a single row would otherwise
// cost as much power, which is what the full chip is short of, as a whole one); more: all of them.
//
// inject(acc, unit) adds values times `unit` to the sums ahead of the last `tail` stages (of all of them if
// there are fewer), and once more, with another unit, if the tile is computed again.
struct SplitNone {
    static constexpr int tail = 0;
    __device__ __forceinline__ void operator()(floatx16 (&)[8], float) const {}
};

template <int LAYOUT, bool SHARED, bool MASK, class Inject = SplitNone>
__device__ __forceinline__ float split_tile(SplitSrc<LAYOUT> &src, SplitLds &L, floatx16 (&acc)[8], float (&csum)[4], int boff,
                                            int rows, int wm, int wn, int tid, const Inject &inject = Inject())
{
    typedef SplitSrc<LAYOUT> Src;
    typedef SplitLds Lds;
    const int lane = tid & 63, lr = lane & 31, lg = lane >> 5;
    const int nstages = src.nstages;
    if (tid == 0) L.redo = 0;

    typename Src::Raw r;
    // Fragment addresses of this lane: column 32 t + lr of a 128-column group sits at 32 j + ((8 t + q) ^ swz) with
    // j = lr & 3, q = lr >> 2; bit 3 of swz is lr & 1, so an even t and the odd one after it need a base each and
    // steps of 16 fragments.
    const int place = ((lr & 3) << 5) | ((lr >> 2) ^ (split_swz(lr & 3) & 7));
    const int odd = (lr & 1) << 3;
    auto tile_at = [&](int t) { return 16 * (t >> 1) + ((8 * (t & 1)) ^ odd); };    // t: 32-column tile of the 128
    const int a0 = lg * Lds::KG_A + wm * 128 + place;
    const int b0 = SHARED ? lg * Lds::KG_A + boff + place : Lds::FRAG_B + lg * Lds::KG_B + place;
    constexpr int pa = S_BM, pb = SHARED ? S_BM : S_BN;      // distance of two pieces of A and of B
    const int fa_e = a0 + tile_at(0), fa_o = a0 + tile_at(1);
    auto fa = [&](int ti) { return ((ti & 1) ? fa_o : fa_e) + 16 * (ti >> 1); };
    const int fb[2] = {b0 + tile_at(2 * wn), b0 + tile_at(2 * wn + 1)};
    // where this thread's columns go (half of a fragment: 8 bytes)
    int wa[LAYOUT == kRows ? 4 : 1], wb[LAYOUT == kRows ? 2 : 1];
    const int kg = src.kq >> 1, half = src.kq & 1;
#pragma unroll
    for (int i = 0; i < (LAYOUT == kRows ? 4 : 1); ++i) wa[i] = 2 * (kg * Lds::KG_A + split_slot(src.col_a(i))) + half;
#pragma unroll
    for (int i = 0; i < (LAYOUT == kRows ? 2 : 1); ++i)
        wb[i] = 2 * (Lds::FRAG_B + kg * Lds::KG_B + split_slot(src.col_b(i))) + half;
    // kNCHW: columns 64 i + cg: 16 i + (cg >> 2) as q, with bit 4 and above free of the swizzle
    auto at_a = [&](int i) { return LAYOUT == kRows ? wa[LAYOUT == kRows ? i : 0] : wa[0] + 2 * ((i & 1) * 16 + (i >> 1) * 128); };
    auto at_b = [&](int i) { return LAYOUT == kRows ? wb[LAYOUT == kRows ? i : 0] : wb[0] + 2 * (i * 16); };

    // Column c of a stage (B's two columns, then A's four) in eight steps: clear what lies past the image, column sum,
    // the three pieces to LDS.
    SplitCut cut;
    auto convert = [&](int c, int step, int valid, suint4 *buf) {
        const bool isa = c >= 2;
        const int i = isa ? c - 2 : c;
        if (!isa && SHARED) return;
        float(&x)[4] = isa ? r.a[isa ? i : 0] : r.b[isa ? 0 : i];
        suint2 *d = reinterpret_cast<suint2 *>(buf) + (isa ? at_a(isa ? i : 0) : at_b(isa ? 0 : i));
        constexpr int piece = 2;                     // halves per fragment
        const int next = piece * (isa ? S_BM : S_BN);
        if (step == 0) {
            if constexpr (LAYOUT == kNCHW && MASK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = 4 * src.kq + e < valid ? x[e] : 0.f;
            }
            if (SHARED) csum[i] += (x[0] + x[1]) + (x[2] + x[3]);
            cut.scale(x);
        } else if (step == 1) {
            cut.half(x, 0, 4);
        } else if (step == 2) {
            cut.top(0, 4);
        } else if (step == 3) {
            d[0] = cut.pack();
            cut.rest(x, 0, 2);
        } else if (step == 4) {
            cut.rest(x, 2, 4);
            cut.half(x, 0, 2);
        } else if (step == 5) {
            cut.half(x, 2, 4);
            cut.top(0, 2);
        } else if (step == 6) {
            cut.top(2, 4);
            d[next] = cut.pack();
        } else {
            cut.rest(x, 0, 4);
            d[2 * next] = cut.pack_last(x);
        }
    };
    auto load_all = [&](const typename Src::At &p) {
        if (!SHARED) src.load_b(r, p);
        src.load_a(r, p);
    };
    auto convert_all = [&](int valid, suint4 *buf) {
#pragma unroll
        for (int c = 0; c < 6; ++c)
#pragma unroll
            for (int step = 0; step < 8; ++step) convert(c, step, valid, buf);
    };

    // Stage g multiplies the fragments of buffer g mod 2 while the values of stage g + 1 are converted into the other
    // one and replaced by loads of stage g + 2.
    int valid = S_KT;                   // of the stage whose values are in r
    auto body = [&](auto rows_c, int g) {
        constexpr int NT = decltype(rows_c)::value;
        const suint4 *buf = L.ring + (g & 1) * Lds::BUF;
        suint4 *out = L.ring + ((g + 1) & 1) * Lds::BUF;
        const typename Src::At p = src.at(g + 2);
        if constexpr (NT > 0) {
            sbf16x8 A[3], B[2][3];
            auto get = [&](int at) { return __builtin_bit_cast(sbf16x8, buf[at]); };
            // in the order of their first use
            A[2] = get(fa(0) + 2 * pa);
            B[0][0] = get(fb[0]);
            B[1][0] = get(fb[1]);
            A[1] = get(fa(0) + pa);
            B[0][1] = get(fb[0] + pb);
            B[1][1] = get(fb[1] + pb);
            A[0] = get(fa(0));
            B[0][2] = get(fb[0] + 2 * pb);
            B[1][2] = get(fb[1] + 2 * pb);
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) {
                // The two column tiles alternate, so that no MFMA waits for the one before it.  A step of the
                // conversion behind every MFMA (the barriers keep the scheduler from gathering them behind the last
                // one).  A piece of A is replaced by that of the next row tile behind its last use.
#pragma unroll
                for (int m = 0; m < 12; ++m) {
                    constexpr int pieceA[6] = {2, 1, 1, 0, 0, 0}, pieceB[6] = {0, 1, 0, 2, 1, 0};
                    const int q = m >> 1, tj = m & 1;
                    acc[2 * ti + tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[pieceA[q]], B[tj][pieceB[q]],
                                                                               acc[2 * ti + tj], 0, 0, 0);
                    if (ti + 1 < NT) {
                        if (m == 1) A[2] = get(fa(ti + 1) + 2 * pa);
                        if (m == 5) A[1] = get(fa(ti + 1) + pa);
                        if (m == 11) A[0] = get(fa(ti + 1));
                    }
                    const int n = 12 * ti + m;
                    if (NT == 4) {
                        convert(n / 8, n % 8, valid, out);
                        if (n == 15 && !SHARED) src.load_b(r, p);
                        if (n == 47) src.load_a(r, p);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (NT < 4) {
            convert_all(valid, out);
            load_all(p);
        }
        valid = p.valid;
        __syncthreads();
    };

#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) csum[i] = 0.f;
    src.rewind();
    {   // stage 0 into the first buffer, stage 1 under way
        typename Src::At p = src.at(0);
        valid = p.valid;
        load_all(p);
        p = src.at(1);
        convert_all(valid, L.ring);
        load_all(p);
        valid = p.valid;
    }
    __syncthreads();
    auto all = [&](auto rows_c) {
        int g = 0;
        if constexpr (Inject::tail > 0) {
            const int at = max(0, nstages - Inject::tail);
            if (nstages == 0) inject(acc, 1.f / kSplitUnscale);
#pragma unroll 1
            for (; g < nstages; ++g) {
                if (g == at) inject(acc, 1.f / kSplitUnscale);
                body(rows_c, g);
            }
        } else {
            for (; g < nstages; ++g) body(rows_c, g);
        }
    };
    if (Inject::tail > 0 || rows > 1) all(std::integral_constant<int, 4>{});      // (with an injection: one way only, or the ways' sums meet in scratch memory)
    else if (rows == 1) all(std::integral_constant<int, 1>{});
    else all(std::integral_constant<int, 0>{});

    // Is every result finite?  Rows and columns past the edge of the operands (a 16-byte piece is not split: they may hold
    // anything) have no say.
    if (rows > 0) {
        int live = src.lim_a - wm * 128 - 4 * lg;            // row 32 ti + 8 (v >> 2) + (v & 3) of this lane exists below this
        float t[2] = {0.f, 0.f};                             // stays 0 unless something is infinite or NaN
#pragma unroll
        for (int ti = 0; ti < 4; ++ti)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if ((v & 3) == 0) asm volatile("" : "+v"(live), "+v"(t[0]), "+v"(t[1]));    // or it keeps 64 masks at once
#pragma unroll
                for (int tj = 0; tj < 2; ++tj)
                    t[tj] = __builtin_fmaf(32 * ti + 8 * (v >> 2) + (v & 3) < live ? acc[2 * ti + tj][v] : 0.f, 0.f, t[tj]);
            }
        const bool finite = (t[0] == 0.f || wn * 64 + lr >= src.lim_b) && (t[1] == 0.f || wn * 64 + 32 + lr >= src.lim_b);
        if (!finite) L.redo = 1;
    }
    __syncthreads();
    if (L.redo == 0) return kSplitUnscale;
    // ---- the fp32 MFMA: rare, written for size ----
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    inject(acc, 1.f);
    float *xs = reinterpret_cast<float *>(L.ring);           // [16 k][columns of A | of B]
    constexpr int XP = S_BM + S_BN + 8;
    src.rewind();
#pragma unroll 1
    for (int g = 0; g < nstages; ++g) {
        const typename Src::At p = src.at(g);
        load_all(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float *row = xs + (4 * src.kq + e) * XP;
#pragma unroll
            for (int i = 0; i < 4; ++i) row[src.col_a(i)] = 4 * src.kq + e < p.valid ? r.a[i][e] : 0.f;
            if (!SHARED) {
#pragma unroll
                for (int i = 0; i < 2; ++i) row[S_BM + src.col_b(i)] = 4 * src.kq + e < p.valid ? r.b[i][e] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int k = lg; k < S_KT; k += 2) {
            const float *row = xs + k * XP + lr;
            const float b0f = row[(SHARED ? boff : S_BM) + wn * 64], b1f = row[(SHARED ? boff : S_BM) + wn * 64 + 32];
#pragma unroll
            for (int ti = 0; ti < 4; ++ti) {
                const float a = row[wm * 128 + 32 * ti];
                acc[2 * ti] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b0f, acc[2 * ti], 0, 0, 0);
                acc[2 * ti + 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b1f, acc[2 * ti + 1], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    return 1.f;
}

}  // namespace kfac
