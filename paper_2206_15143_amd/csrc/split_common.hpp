// The split-fp16 product core shared by gemm_split.hpp and syrk_split.hpp: tiles of C = A^T B for fp32 operands on
// the fp16 MFMA units, at fp32 accuracy.
//
// Arithmetic.  A column of an operand (the index that is not contracted) is scaled by a power of two s, exact, and
// every scaled value is cut into two fp16 pieces, h = fp16(s x) and l = fp16(s x - h), both rounded to nearest.
// |s x - h| is at most half an ulp of 11 bits and a multiple of the last bit of x, i.e. a 12-bit number, of which l
// keeps 11: x = (h + l) / s up to one unit in the last place of the fp32 value, 2^-23 |x|, and exactly for three
// values in four.  The product keeps
//     a b  ~  ( ah bh + ah bl + al bh ) / (sa sb),
// each term exact in the fp32 accumulator of v_mfma_f32_32x32x16_f16.  The term left out, al bl, is below 2^-22 |a b|
// and as often positive as negative: with the two roundings of the operands the error of a product is at most
// 2^-21 |a b|.  (The cut into three truncated bf16 pieces and six products that this replaced has the same bound
// from the terms it leaves out, all of one sign: a2 b3 + a3 b2 <= 2 * 2^-7 * 2^-15 |a b|.)  Half the MFMA
// instructions and a fifth of the conversion work.
//
// Range.  fp16 has 5 exponent bits, hence the scale.  It is taken per column from the first K stage of the tile (and,
// for the matrices of a product, from the diagonal element: half of the operands here are inverses, whose columns
// have their largest element there), so that the largest value seen lands in [2^8, 2^9): 64 times larger ones may
// follow.  A column of zeros is given the scale of the whole operand.  While the tile runs every thread keeps the true
// maxima of the columns it loads; at the end a column whose maximum left [2^4, 2^15) makes the workgroup compute the
// tile once more, with the maxima now known.  A value of a column therefore carries an error of one fp32 ulp or of
// 2^-25 / 2^4 = 2^-29 (as a rule 2^-33) of the column's maximum, whichever is larger.  The second kind is far below the
// rounding of the sum unless the large values of one operand only ever meet tiny values of the other: a tile in which
// more than a quarter of a wavefront's columns have no result of 2^19 times what these errors can add up to is
// computed on the fp32 MFMA instead.
//
// Pipeline.  A workgroup of four wavefronts owns a tile of 64 NTI x 128 (NTI = 4 or 2), a wavefront half of the rows
// and half of the columns.  K goes in stages of 16 rows = one MFMA step.  A thread loads four k of NTI columns of A and
// of two of B, with 16- and 8-byte loads (a load instruction costs a wavefront about 16 cycles of the address unit
// whatever its width: with 4-byte loads that unit bounded the kernel, 2.1 us per stage and CU), three stages ahead.
// The values are converted ONCE per workgroup and written to LDS as halves of ready fragments (a fragment = the eight
// k of one column and piece = 16 bytes) in a ring of three buffers, one barrier per stage.  The conversion (three VALU
// operations per value and half of one for the maxima) runs between the MFMAs, four operations beside each of the 24
// of a wavefront.  Fragments of consecutive columns are spread over LDS by split_slot so that the MFMA reads (32
// consecutive columns) and the writes (every fourth column) both touch every bank group equally.
#pragma once

#include <type_traits>

#include "wave_common.hpp"

namespace kfac {

constexpr int S_BM = 256;                     // rows of C per workgroup (columns of A) of the large tile
constexpr int S_BN = 128;                     // columns of C per workgroup (columns of B)
constexpr int S_KT = 16;                      // rows of the operands per stage

typedef _Float16 shalf8 __attribute__((ext_vector_type(8)));
typedef unsigned suint4 __attribute__((ext_vector_type(4)));
typedef unsigned suint2 __attribute__((ext_vector_type(2)));
typedef int sint4 __attribute__((ext_vector_type(4)));
typedef int sint2 __attribute__((ext_vector_type(2)));

// The conversion of four values, in three steps that the K loop spreads over its MFMAs: scale, high pieces, low
// pieces.  (v_fma_mixlo_f16 would scale, round and pack in one instruction, but takes twice the issue slots of these
// and does not run beside an MFMA.)
typedef float sfloat2 __attribute__((ext_vector_type(2)));
typedef _Float16 shalf2 __attribute__((ext_vector_type(2)));
struct SplitConv {
    sfloat2 u[2];
    shalf2 h[2], l[2];
    __device__ __forceinline__ void scale(const float (&x)[4], float s)
    {
        u[0] = sfloat2{x[0] * s, x[1] * s};
        u[1] = sfloat2{x[2] * s, x[3] * s};
    }
    __device__ __forceinline__ void high()
    {
        h[0] = __builtin_convertvector(u[0], shalf2);          // v_cvt_pk_f16_f32
        h[1] = __builtin_convertvector(u[1], shalf2);
    }
    // x s - h: one v_fma_mix_f32 each, exact
    __device__ __forceinline__ sfloat2 rest(const float (&x)[4], float s, int q) const
    {
        return sfloat2{__builtin_fmaf(x[2 * q], s, -(float)h[q].x), __builtin_fmaf(x[2 * q + 1], s, -(float)h[q].y)};
    }
};
// max(m, |a|, |b|)
__device__ __forceinline__ float split_max3(float m, float a, float b)
{
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
    return m;
}

// exponent field of the power of two that brings a maximum m (bit pattern of a value >= 0) into [2^t, 2^(t+1))
__device__ __forceinline__ int split_scale_exp(unsigned m, int t)
{
    const int e = 254 + t - (int)(m >> 23);
    return e < 1 ? 1 : (e > 254 ? 254 : e);
}

// Place of column c (of up to 256) among the fragments of one k group and piece: groups of 128 columns, inside them
// column 4 q + j goes to 32 j + (q ^ swizzle(j)).
__host__ __device__ constexpr int split_swz(int j) { return ((j & 1) << 3) | ((j >> 1) << 2) | ((j & 1) << 1); }
__device__ __forceinline__ int split_slot(int c)
{
    return (c & ~127) | ((c & 3) << 5) | (((c & 127) >> 2) ^ split_swz(c & 3));
}

// LDS of a workgroup: the stage buffers of fragments, the scale exponents, the column maxima and a flag word
template <int NTI>
struct SplitLds {
    static constexpr int BM = 64 * NTI;
    static constexpr int KG_A = 2 * BM + 1;                  // fragments from k group 0 to 1 (both pieces; odd: see split_tile)
    static constexpr int KG_B = 2 * S_BN + 1;
    static constexpr int FRAG_B = 2 * KG_A;                  // first fragment of B
    static constexpr int BUF = 2 * KG_A + 2 * KG_B;          // fragments per stage buffer
    static constexpr int EPI = 4 * 32 * 68 / 4;              // the epilogue's chunks, in 16-byte units
    static constexpr int RING = 3 * BUF > EPI ? 3 * BUF : EPI;
    suint4 ring[RING];
    int ex[BM + S_BN];                                       // exponents of the scales, minus the bias
    unsigned mx[BM + S_BN + 2];                              // maxima of A's and B's columns, of all of A, all of B
    unsigned top[2];                                         // largest scaled maximum of A's columns, per half of the rows
    int redo;
};

// Where the operands of a tile come from, and which part of a stage a thread handles: four k (quarter kq of the
// stage) of the columns col_a(0 .. NTI - 1) of A and col_b(0 .. 1) of B.
// kRows: element (k, c) at base + k ld + c.  The columns of a thread are neighbours: one load instruction per row.
// kNCHW: element (k = n hw + p, c) at (n ctot + c) hw + p; a stage never crosses an image.  The four k are
// neighbours: one 16-byte load per column, four neighbouring lanes the 16 positions of a channel.
template <int NTI, int LAYOUT>
struct SplitSrc {
    __amdgpu_buffer_rsrc_t ra, rb;
    unsigned va[LAYOUT == kRows ? 1 : NTI], vb[LAYOUT == kRows ? 1 : 2];   // byte offset of the column(s), or W_OOB
    unsigned lda4, ldb4;           // kRows: row pitch in bytes
    int lim_a, lim_b;              // columns of the tile that exist
    int diag_a, diag_b, rows;      // kRows: row of the diagonal element of column 0 of the tile, and the number of rows
    unsigned off_a, off_b;         // ... byte offset of column 0
    int nstages;
    int hw, tpi, img0, kt0, ii, ik;   // kNCHW: image walk
    unsigned img_bytes;
    int cg, kq;                    // this thread's column group (0 .. 63) and quarter of the stage

    struct Raw {
        float a[NTI][4], b[2][4];  // [column][k]
    };

    __device__ __forceinline__ void init_thread(int tid)
    {
        const int lane = tid & 63, w = tid >> 6;
        cg = 16 * w + (LAYOUT == kRows ? (lane >> 1) & 15 : lane >> 2);
        kq = LAYOUT == kRows ? 2 * (lane >> 5) + (lane & 1) : lane & 3;
    }
    __device__ __forceinline__ int col_a(int i) const { return LAYOUT == kRows ? NTI * cg + i : 64 * i + cg; }
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
            p.sa = p.live ? (unsigned)(g * S_KT) * lda4 : 0u;
            p.sb = p.live ? (unsigned)(g * S_KT) * ldb4 : 0u;
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
            load_rows<NTI>(r.a, ra, in(p) ? va[0] : W_OOB, p.sa, p.live ? lda4 : 0u);
        } else {
#pragma unroll
            for (int i = 0; i < NTI; ++i) load_pos(r.a[i], ra, in(p) ? va[i] : W_OOB, p.sa);
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

// The K loop of a tile.  acc: 2 NTI accumulator tiles, [ti][tj], of the wavefront's 32 NTI x 64 part, still scaled:
// the value is acc * 2^-(ex[row] + ex[BM + column]) with the exponents left in L.ex.  SHARED: B's columns are columns
// boff .. boff + 127 of A (tiles on the diagonal of X^T X; boff is 0 or 128): B is neither loaded nor converted, and
// the sums of this thread's columns of A over its k go to csum.  MASK: some NCHW problem of the launch has a number
// of positions that is no multiple of 4 (positions past the end of an image hold the next channel's data).
// `rows`: row tiles (of 32 rows) of the wavefront's part that are wanted.  0: it only helps with the staging; 1: it
// multiplies that one (the bias column makes orders of 2^n + 1 the rule here: a tile for a single row would otherwise
// cost as much power, which is what the full chip is short of, as a whole one); more: all of them.
template <int NTI, int LAYOUT, bool SHARED, bool MASK>
__device__ __forceinline__ void split_tile(SplitSrc<NTI, LAYOUT> &src, SplitLds<NTI> &L, floatx16 (&acc)[2 * NTI],
                                           float (&csum)[NTI], int boff, int rows, int wm, int wn, int tid)
{
    typedef SplitSrc<NTI, LAYOUT> Src;
    typedef SplitLds<NTI> Lds;
    constexpr int BM = Lds::BM;
    const int lane = tid & 63, lr = lane & 31, lg = lane >> 5;
    const int nstages = src.nstages;
    float sA[NTI], sB[2], mA[NTI], mB[2];

    for (int e = tid; e < BM + S_BN + 2; e += 256) L.mx[e] = 0u;
    if (tid == 0) L.redo = 0;
    if (tid < 2) L.top[tid] = 0u;
    __syncthreads();

    typename Src::Raw r;
    // Fragment addresses of this lane: column 32 t + lr of a 128-column group sits at 32 j + ((8 t + q) ^ swz) with
    // j = lr & 3, q = lr >> 2; bit 3 of swz is lr & 1, so an even t and the odd one after it need a base each and
    // steps of 16 fragments.
    const int place = ((lr & 3) << 5) | ((lr >> 2) ^ (split_swz(lr & 3) & 7));
    const int odd = (lr & 1) << 3;
    const int a0 = lg * Lds::KG_A + (NTI == 4 ? wm * 128 : 0) + place;
    const int b0 = SHARED ? lg * Lds::KG_A + boff + place : Lds::FRAG_B + lg * Lds::KG_B + place;
    constexpr int pb = SHARED ? BM : S_BN;            // distance of B's two pieces
    auto tile_at = [&](int t) { return 16 * (t >> 1) + ((8 * (t & 1)) ^ odd); };    // t: 32-column tile of the 128
    const int ta0 = NTI == 4 ? 0 : 2 * wm, tb0 = 2 * wn;
    const int fa_e = a0 + tile_at(ta0), fa_o = a0 + tile_at(ta0 + 1);
    auto fa = [&](int ti) { return ((ti & 1) ? fa_o : fa_e) + 16 * (ti >> 1); };
    const int fb_e = b0 + tile_at(tb0), fb_o = b0 + tile_at(tb0 + 1);
    // where this thread's columns go (half of a fragment: 8 bytes)
    int wa[LAYOUT == kRows ? NTI : 1], wb[LAYOUT == kRows ? 2 : 1];
    const int kg = src.kq >> 1, half = src.kq & 1;
#pragma unroll
    for (int i = 0; i < (LAYOUT == kRows ? NTI : 1); ++i) wa[i] = 2 * (kg * Lds::KG_A + split_slot(src.col_a(i))) + half;
#pragma unroll
    for (int i = 0; i < (LAYOUT == kRows ? 2 : 1); ++i)
        wb[i] = 2 * (Lds::FRAG_B + kg * Lds::KG_B + split_slot(src.col_b(i))) + half;
    // kNCHW: columns 64 i + cg: 16 i + (cg >> 2) as q, with bit 4 and above free of the swizzle
    auto at_a = [&](int i) { return LAYOUT == kRows ? wa[LAYOUT == kRows ? i : 0] : wa[0] + 2 * ((i & 1) * 16 + (i >> 1) * 128); };
    auto at_b = [&](int i) { return LAYOUT == kRows ? wb[LAYOUT == kRows ? i : 0] : wb[0] + 2 * (i * 16); };

    auto mask4 = [&](float (&x)[4], int valid) {
        if constexpr (LAYOUT == kNCHW && MASK) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = 4 * src.kq + e < valid ? x[e] : 0.f;
        }
    };
    auto maxima = [&](int valid) {
#pragma unroll
        for (int i = 0; i < NTI; ++i) {
            mask4(r.a[i], valid);
            mA[i] = split_max3(split_max3(mA[i], r.a[i][0], r.a[i][1]), r.a[i][2], r.a[i][3]);
        }
        if (!SHARED) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mask4(r.b[i], valid);
                mB[i] = split_max3(split_max3(mB[i], r.b[i][0], r.b[i][1]), r.b[i][2], r.b[i][3]);
            }
        }
    };
    // Column c of a stage (A's NTI columns, then B's two) in three steps: clear what lies past the image, maximum,
    // column sum, scale | high pieces | low pieces, both to LDS.
    SplitConv cv;
    auto convert = [&](int c, int step, int valid, suint4 *buf) {
        const bool isa = c < NTI;
        const int i = isa ? c : c - NTI;
        if (!isa && SHARED) return;
        float(&x)[4] = isa ? r.a[isa ? i : 0] : r.b[isa ? 0 : i];
        const float s = isa ? sA[isa ? i : 0] : sB[isa ? 0 : i];
        if (step == 0) {
            float &m = isa ? mA[isa ? i : 0] : mB[isa ? 0 : i];
            mask4(x, valid);
            m = split_max3(split_max3(m, x[0], x[1]), x[2], x[3]);
            if (SHARED) csum[i] += (x[0] + x[1]) + (x[2] + x[3]);
            cv.scale(x, s);
        } else if (step == 1) {
            cv.high();
            cv.u[0] = cv.rest(x, s, 0);
        } else {
            cv.u[1] = cv.rest(x, s, 1);
            cv.l[0] = __builtin_convertvector(cv.u[0], shalf2);
            cv.l[1] = __builtin_convertvector(cv.u[1], shalf2);
            suint2 *d = reinterpret_cast<suint2 *>(buf) + (isa ? at_a(isa ? i : 0) : at_b(isa ? 0 : i));
            d[0] = suint2{__builtin_bit_cast(unsigned, cv.h[0]), __builtin_bit_cast(unsigned, cv.h[1])};
            d[2 * (isa ? BM : S_BN)] = suint2{__builtin_bit_cast(unsigned, cv.l[0]), __builtin_bit_cast(unsigned, cv.l[1])};
        }
    };
    auto load_all = [&](const typename Src::At &p) {
        src.load_a(r, p);
        if (!SHARED) src.load_b(r, p);
    };
    auto convert_all = [&](int valid, suint4 *buf) {
#pragma unroll
        for (int c = 0; c < NTI + 2; ++c)
#pragma unroll
            for (int step = 0; step < 3; ++step) convert(c, step, valid, buf);
    };

    // Stage g multiplies the fragments of buffer g mod 3 while the values of stage g + 2 are converted into buffer
    // (g + 2) mod 3 and, task by task, replaced by loads of stage g + 3.  Buffer (g + 1) mod 3 was complete at the last
    // barrier: the first fragments of stage g + 1 are read before the barrier at the end of stage g, so that no
    // wavefront starts a stage with the latency of LDS.
    int rd, nx, wr;                     // buffers of stages g, g + 1, g + 2
    int valid = S_KT;                   // of the stage whose values are in r
    auto body = [&](auto rows_c, int g, shalf8 (&B)[4], suint4 &ah, suint4 &al) {
        constexpr int NT = decltype(rows_c)::value;
        suint4 *out = L.ring + wr;
        const typename Src::At p = src.at(g + 3);
        if constexpr (NT > 0) {
            const suint4 *buf = L.ring + rd, *next = L.ring + nx;
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) {
                const shalf8 A1 = __builtin_bit_cast(shalf8, ah), A2 = __builtin_bit_cast(shalf8, al);
                if (ti + 1 < NT) {
                    ah = buf[fa(ti + 1)];
                    al = buf[fa(ti + 1) + BM];
                } else {
                    ah = next[fa(0)];
                    al = next[fa(0) + BM];
                }
                // Small terms first; the two column tiles alternate, so that no MFMA waits for the one before it.  A
                // step of the conversion behind every MFMA (the barriers keep the scheduler from gathering them
                // behind the last one), the loads of A once its columns are converted, then those of B.
#pragma unroll
                for (int m = 0; m < 6; ++m) {
                    const shalf8 am = m < 2 ? A2 : A1;
                    const shalf8 bm = B[(m & 1) * 2 + (m == 2 || m == 3 ? 1 : 0)];
                    acc[2 * ti + (m & 1)] = __builtin_amdgcn_mfma_f32_32x32x16_f16(am, bm, acc[2 * ti + (m & 1)], 0, 0, 0);
                    const int n = 6 * ti + m;
                    if (NT == NTI) {
                        if (n < 3 * (NTI + 2)) convert(n / 3, n % 3, valid, out);
                        if (n == 3 * NTI) src.load_a(r, p);
                        if (n == (NTI == 4 ? 3 * NTI + 6 : 11) && !SHARED) src.load_b(r, p);
                    }
                    // B of the next stage, each fragment behind its last use
                    if (ti == NT - 1 && m == 2) B[1] = __builtin_bit_cast(shalf8, next[fb_e + pb]);
                    if (ti == NT - 1 && m == 3) B[3] = __builtin_bit_cast(shalf8, next[fb_o + pb]);
                    if (ti == NT - 1 && m == 4) B[0] = __builtin_bit_cast(shalf8, next[fb_e]);
                    if (ti == NT - 1 && m == 5) B[2] = __builtin_bit_cast(shalf8, next[fb_o]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (NT < NTI) {
            convert_all(valid, out);
            load_all(p);
        }
        valid = p.valid;
        const int free_buf = rd;
        rd = nx; nx = wr; wr = free_buf;
        __syncthreads();
    };
    auto k_loop = [&](auto rows_c) {
        shalf8 B[4];
        suint4 ah, al;
        if constexpr (decltype(rows_c)::value > 0) {
            B[0] = __builtin_bit_cast(shalf8, L.ring[fb_e]);
            B[1] = __builtin_bit_cast(shalf8, L.ring[fb_e + pb]);
            B[2] = __builtin_bit_cast(shalf8, L.ring[fb_o]);
            B[3] = __builtin_bit_cast(shalf8, L.ring[fb_o + pb]);
            ah = L.ring[fa(0)];
            al = L.ring[fa(0) + BM];
        }
        for (int g = 0; g < nstages; ++g) body(rows_c, g, B, ah, al);
    };

    for (int attempt = 0;; ++attempt) {
#pragma unroll
        for (int i = 0; i < 2 * NTI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
#pragma unroll
        for (int i = 0; i < NTI; ++i) mA[i] = csum[i] = 0.f;
        mB[0] = mB[1] = 0.f;
        src.rewind();
        rd = 0; nx = Lds::BUF; wr = 2 * Lds::BUF;
        typename Src::At p = src.at(0);
        valid = p.valid;
        load_all(p);
        // this thread's maxima into the table (an integer maximum: the bits of values >= 0 order alike); columns past
        // the edge of the operand may hold anything and have no say
        auto publish = [&]() {
#pragma unroll
            for (int i = 0; i < NTI; ++i)
                if (src.col_a(i) < src.lim_a) atomicMax(&L.mx[src.col_a(i)], __float_as_uint(mA[i]));
            if (!SHARED) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (src.col_b(i) < src.lim_b) atomicMax(&L.mx[BM + src.col_b(i)], __float_as_uint(mB[i]));
            }
        };
        if (attempt == 0) {
            if constexpr (LAYOUT == kRows && !SHARED) {
                for (int e = tid; e < BM + S_BN; e += 256) {
                    const bool isa = e < BM;
                    const int c = isa ? e : e - BM, row = (isa ? src.diag_a : src.diag_b) + c;
                    const bool there = row >= 0 && row < src.rows && c < (isa ? src.lim_a : src.lim_b);
                    const unsigned o = (unsigned)row * (isa ? src.lda4 : src.ldb4) + (isa ? src.off_a : src.off_b) + 4u * (unsigned)c;
                    const unsigned x = isa ? __builtin_amdgcn_raw_buffer_load_b32(src.ra, there ? o : W_OOB, 0, 0)
                                           : __builtin_amdgcn_raw_buffer_load_b32(src.rb, there ? o : W_OOB, 0, 0);
                    atomicMax(&L.mx[e], x & 0x7fffffffu);
                }
            }
            maxima(valid);
            publish();
            float ta = 0.f, tb = 0.f;
#pragma unroll
            for (int i = 0; i < NTI; ++i) ta = fmaxf(ta, src.col_a(i) < src.lim_a ? mA[i] : 0.f);
#pragma unroll
            for (int i = 0; i < 2; ++i) tb = fmaxf(tb, src.col_b(i) < src.lim_b ? mB[i] : 0.f);
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                ta = fmaxf(ta, __shfl_xor(ta, off));
                tb = fmaxf(tb, __shfl_xor(tb, off));
            }
            if (lane == 0) {
                atomicMax(&L.mx[BM + S_BN], __float_as_uint(ta));
                atomicMax(&L.mx[BM + S_BN + 1], __float_as_uint(tb));
            }
            __syncthreads();
        }
        // the scales: from the maximum of the column, or, of a column of zeros, of the whole operand
        auto scale_of = [&](int slot, int whole) {
            unsigned m = L.mx[slot];
            if (m == 0u) m = L.mx[whole];
            return split_scale_exp(m, attempt == 0 ? 8 : 13);
        };
        for (int e = tid; e < BM + (SHARED ? 0 : S_BN); e += 256)
            L.ex[e] = scale_of(e, e < BM ? BM + S_BN : BM + S_BN + 1) - 127;
#pragma unroll
        for (int i = 0; i < NTI; ++i) sA[i] = __uint_as_float((unsigned)scale_of(src.col_a(i), BM + S_BN) << 23);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            sB[i] = SHARED ? 1.f : __uint_as_float((unsigned)scale_of(BM + src.col_b(i), BM + S_BN + 1) << 23);
        // stages 0 and 1 into the first two buffers, stage 2 under way
#pragma unroll 1
        for (int st = 0; st < 2; ++st) {
            p = src.at(st + 1);
            convert_all(valid, L.ring + st * Lds::BUF);
            load_all(p);
            valid = p.valid;
        }
        __syncthreads();
        if (rows > 1) k_loop(std::integral_constant<int, NTI>{});
        else if (rows == 1) k_loop(std::integral_constant<int, 1>{});
        else k_loop(std::integral_constant<int, 0>{});
        if (attempt == 1) break;
        // did the scales hold?  (the maxima only grow, so the table takes the final ones on top of the first stage's)
        publish();
        __syncthreads();
        bool bad = false;
        for (int e = tid; e < BM + (SHARED ? 0 : S_BN); e += 256) {
            const unsigned m = L.mx[e];
            const int top = (int)(m >> 23) + L.ex[e];        // exponent field of the scaled maximum
            // the clamped scales of subnormal or huge columns are as good as they get
            const int se = L.ex[e] + 127;
            if (m != 0u && ((top > 127 + 14 && se > 1) || (top < 127 + 4 && se < 254))) bad = true;
        }
        if (bad) L.redo = 1;
        __syncthreads();
        if (L.redo == 0) break;      // uniform: the word is not written again before the next barrier
    }
    if (SHARED) {
        // B's scales and maxima are A's
        for (int e = tid; e < S_BN; e += 256) {
            L.ex[BM + e] = L.ex[boff + e];
            L.mx[BM + e] = L.mx[boff + e];
        }
    }
    for (int e = tid; e < BM; e += 256)
        atomicMax(&L.top[e / (BM / 2)], __float_as_uint(ldexpf(__uint_as_float(L.mx[e]), L.ex[e])));
    __syncthreads();
    if (rows > 0) {
        // the largest result of a column against K (2^-25 of the largest scaled values that the other operand offers)
        const float ma = __uint_as_float(L.top[wm]);
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
            float m = 0.f;
#pragma unroll
            for (int ti = 0; ti < NTI; ++ti)
#pragma unroll
                for (int v = 0; v < 16; v += 2) m = split_max3(m, acc[2 * ti + tj][v], acc[2 * ti + tj][v + 1]);
            m = fmaxf(m, __shfl_xor(m, 32));
            const int c = BM + wn * 64 + tj * 32 + lr;
            const float mb = ldexpf(__uint_as_float(L.mx[c]), L.ex[c]);
            const bool weak = m > 0.f && m < (float)nstages * (S_KT / 64.f) * (ma + mb);
            if (__popcll(__ballot(weak)) > 16) L.redo = 2;
        }
    }
    __syncthreads();
    if (L.redo != 2) return;
    // ---- the fp32 MFMA: rare, written for size ----
    for (int e = tid; e < BM + S_BN; e += 256) L.ex[e] = 0;
#pragma unroll
    for (int i = 0; i < 2 * NTI; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    float *xs = reinterpret_cast<float *>(L.ring);           // [16 k][columns of A | of B]
    constexpr int XP = BM + S_BN + 8;
    src.rewind();
#pragma unroll 1
    for (int g = 0; g < nstages; ++g) {
        const typename Src::At p = src.at(g);
        load_all(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float *row = xs + (4 * src.kq + e) * XP;
#pragma unroll
            for (int i = 0; i < NTI; ++i) row[src.col_a(i)] = 4 * src.kq + e < p.valid ? r.a[i][e] : 0.f;
            if (!SHARED) {
#pragma unroll
                for (int i = 0; i < 2; ++i) row[BM + src.col_b(i)] = 4 * src.kq + e < p.valid ? r.b[i][e] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int k = lg; k < S_KT; k += 2) {
            const float *row = xs + k * XP + lr;
            const float b0 = row[(SHARED ? boff : BM) + wn * 64], b1 = row[(SHARED ? boff : BM) + wn * 64 + 32];
#pragma unroll
            for (int ti = 0; ti < NTI; ++ti) {
                const float a = row[wm * (BM / 2) + 32 * ti];
                acc[2 * ti] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b0, acc[2 * ti], 0, 0, 0);
                acc[2 * ti + 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b1, acc[2 * ti + 1], 0, 0, 0);
            }
        }
        __syncthreads();
    }
}

// exponents by which the accumulators of row tile ti have to be multiplied: row r of the tile is 8 q + 4 lg + e
// (accumulator register 4 q + e)
template <int NTI>
__device__ __forceinline__ void split_unscale(floatx16 &c, const SplitLds<NTI> &L, int row0, int col, int lg)
{
    const int en = L.ex[SplitLds<NTI>::BM + col];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const sint4 em = *reinterpret_cast<const sint4 *>(&L.ex[row0 + 8 * q + 4 * lg]);
#pragma unroll
        for (int e = 0; e < 4; ++e) c[4 * q + e] = ldexpf(c[4 * q + e], -(em[e] + en));
    }
}

}  // namespace kfac
