// The triangular inverse of a 16 x 16 block in the registers of one wavefront (the diagonal blocks of invert_chol.hpp, the pivot
// blocks of invert_fused.hpp).
#pragma once

#include "wave_common.hpp"

namespace kfac {

// Lane (q, n) of the result: lane (G, n) of x[q].
template <int G>
__device__ __forceinline__ float chol_rows(const floatx4 &x)
{
    auto u = [](float f) { return __float_as_uint(f); };
    const auto h0 = __builtin_amdgcn_permlane32_swap(u(x[0]), u(x[2]), false, false);
    const auto h1 = __builtin_amdgcn_permlane32_swap(u(x[1]), u(x[3]), false, false);
    const auto g = __builtin_amdgcn_permlane16_swap(G & 2 ? h0[1] : h0[0], G & 2 ? h1[1] : h1[0], false, false);
    return __uint_as_float(G & 1 ? g[1] : g[0]);
}

// Pivots 4 G .. 4 G + 3 of the 16 x 16 block t (MFMA result layout) and of e, which was the identity.  The four rows lie in the
// same lanes, one register each: they are eliminated there; what they take away from the rows behind them is one MFMA each.
template <int G>
__device__ __forceinline__ void chol_pivots(floatx4 &t, floatx4 &e, floatx4 &pivot, int lq, int ln)
{
    const bool own = lq == G;
    float r[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        auto lane_of = [&](int v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t[p]), 20 * G + v)); };
        const float d = lane_of(p);
        float s[4];
#pragma unroll
        for (int v = p + 1; v < 4; ++v) s[v] = lane_of(v);
        float c = __builtin_amdgcn_rcpf(d);
        c = __builtin_fmaf(__builtin_fmaf(-d, c, 1.f), c, c);
        r[p] = d > 0.f && d < 0x1p126f ? -c : 0.f;
        pivot[p] = own ? d : pivot[p];
        const float mine = own ? r[p] : 0.f;
#pragma unroll
        for (int v = p + 1; v < 4; ++v) {
            const float m = s[v] * mine;
            t[v] = __builtin_fmaf(m, t[p], t[v]);
            e[v] = __builtin_fmaf(m, e[p], e[v]);
        }
    }
    if constexpr (G < 3) {
        const float bt = chol_rows<G>(t), be = chol_rows<G>(e);
        const float rq = lq < 2 ? (lq == 0 ? r[0] : r[1]) : (lq == 2 ? r[2] : r[3]);
        const float at = ln >= 4 * (G + 1) ? bt * rq : 0.f;
        e = __builtin_amdgcn_mfma_f32_16x16x4f32(at, be, e, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x4f32(at, bt, t, 0, 0, 0);
    }
}

// X of the 16 x 16 block t (MFMA result layout, from the diagonal up), one wavefront; rows are scaled at the end, so that a
// pivot waits for one reciprocal and a few multiply-adds of the one before it.  A pivot that is not positive leaves a
// zero row and is reported: 1-based place in the block, or 0.  fix: 1 / pivot less the square of its rounded root.
__device__ __forceinline__ int chol_leaf(floatx4 &t, floatx4 &fix, int lane)
{
    const int lq = lane >> 4, ln = lane & 15;
    floatx4 e, pivot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 4; ++v) e[v] = 4 * lq + v == ln ? 1.f : 0.f;
    chol_pivots<0>(t, e, pivot, lq, ln);
    chol_pivots<1>(t, e, pivot, lq, ln);
    chol_pivots<2>(t, e, pivot, lq, ln);
    chol_pivots<3>(t, e, pivot, lq, ln);
    int fail = 0;
#pragma unroll
    for (int v = 3; v >= 0; --v) {
        // 1 / sqrt(pivot), the instruction's last bit corrected
        const float p = pivot[v];
        float r = __builtin_amdgcn_rsqf(p);
        const float h = p * r, c = __builtin_fmaf(-__builtin_fmaf(p, r, -h), r, __builtin_fmaf(-h, r, 1.f));
        r = __builtin_fmaf(0.5f * r, c, r);
        const bool ok = p > 0.f, kept = ok && p < 0x1p126f;
        t[v] = e[v] * (kept ? r : 0.f);
        const float g = p * r, l = __builtin_fmaf(-__builtin_fmaf(p, r, -g), r, __builtin_fmaf(-g, r, 1.f));
        fix[v] = kept ? l * r * r : 0.f;
        fail = ok ? fail : 4 * lq + v + 1;
    }
    int first = 0;
#pragma unroll
    for (int q = 3; q >= 0; --q) {
        const int f = __builtin_amdgcn_readlane(fail, 16 * q);
        first = f != 0 ? f : first;
    }
    return first;
}

}  // namespace kfac
