// Two-sided products  P = G^T W A  of narrow layers in one launch: the preconditioning of Eq. 5 of the DP-KFAC paper
// (A = A_inv, G = G_inv, both symmetric) and either half of Eq. 13 (A = Q_A, G = Q_G with the division in the epilogue,
// then their transposes), for layers one of whose dimensions is at most 64.
//
// Bound: for a network of narrow layers (110 layers of a ResNet-110, orders 145 to 577) neither flops nor bytes but the
// chain K loop - store - launch - K loop of the two products of every layer, walked by few wavefronts.  So:
//   - the products are associated so that the deep one comes first and its result stays on the chip: with d_G <= 64 a
//     workgroup owns 16 TN columns of P and forms T = W A[:, tile] (K = d_A), then G^T T (K = d_G); with d_A <= 64 it owns
//     16 TN rows and forms (W^T G[:, tile])^T, then that times A.  No intermediate in memory, nothing is computed twice.
//   - the wavefronts of a workgroup split K among them (chunks of 16 in turn) and every wavefront computes the whole
//     tile: operands go from memory to registers in the layout the MFMA wants, 16 bytes per lane, with no LDS and no
//     barrier in the loop.  Of the operand whose rows are contiguous along the tile a lane takes TN (MT) neighbouring
//     columns, which become the same column of TN (MT) interleaved MFMA tiles; of W, contiguous along K, four
//     neighbouring k, which become its elements of four MFMA steps.
//   - the parts are added in wavefront order through LDS, wavefront t taking MFMA tile t: the sums land in the very
//     registers the second product reads as its operand.
// 110 layers of the ResNet-110 shape: 14 + 48 us as two launches of 64-wide block tiles with all wavefronts on one K stage,
// now 33 us (one million MFMAs: 13 us of the matrix units), the call 58 -> 30 us with the operands in the last-level cache
// and 68 -> 48 with them in memory (two chunks of loads in flight per wavefront).
#include "common.hpp"

#include <algorithm>
#include <vector>

namespace kfac {

namespace {

constexpr int kMaxPrec = 128;     // layers per launch (a 9 KB kernel argument)

struct PrecProb {
    const float *W, *A, *G;
    float *out;
    const float *rv, *cv;         // null, or the eigenvalues of the division (out rows, out columns)
    int dA, dG;
    int tiles;
    int var;                      // MT - 1, plus 4 when d_A is the small dimension
};

struct PrecTable {
    int count;
    int group_blk[kMaxPrec / 8 + 1];   // first block of every group of eight layers
    int rest_blk[8];              // first block of the layers of the last, incomplete group
    float gamma;
    PrecProb p[kMaxPrec];
};

typedef int pint4 __attribute__((ext_vector_type(4)));
typedef int pint2 __attribute__((ext_vector_type(2)));

// N neighbouring floats; what lies past the end of the buffer reads as zero, every element by itself
template <int N>
__device__ __forceinline__ void load_n(float (&x)[N], __amdgpu_buffer_rsrc_t r, unsigned off)
{
    if constexpr (N == 4) {
        const pint4 v = __builtin_bit_cast(pint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __int_as_float(v[e]);
    } else if constexpr (N == 2) {
        const pint2 v = __builtin_bit_cast(pint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
        x[0] = __int_as_float(v[0]);
        x[1] = __int_as_float(v[1]);
    } else {
        x[0] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    }
}

// One tile of one layer.  MT: 16-wide MFMA tiles of the small dimension; ROWS: d_G is the small one (W is read along
// its rows), else d_A.  LDS: the parts of the other wavefronts, then the tile on its way out.
template <int MT, int TN, int NW, bool ROWS>
__device__ __forceinline__ void precond_tile(const PrecProb &pr, int tile, float gamma, floatx4 *lds)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int S = ROWS ? pr.dG : pr.dA;          // small dimension
    const int L = ROWS ? pr.dA : pr.dG;          // the dimension that is cut into tiles, and the depth of the first product
    const int n0 = tile * 16 * TN;
    const float *Yp = ROWS ? pr.A : pr.G, *Zp = ROWS ? pr.G : pr.A;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(pr.W), 0, pr.dA * pr.dG * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Yp), 0, L * L * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Zp), 0, S * S * 4, 0x00020000);

    // row of the small dimension that register v of MFMA tile i holds
    auto row_of = [&](int i, int v) { return ROWS ? 16 * i + 4 * lk + v : MT * (4 * lk + v) + i; };

    floatx4 acc[MT][TN];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};

    struct Chunk {
        float a[ROWS ? MT : 4][ROWS ? 4 : MT];
        float b[4][TN];
    };
    auto load = [&](Chunk &c, int ch) {
        const int k = 16 * ch + 4 * lk;
#pragma unroll
        for (int e = 0; e < 4; ++e) load_n<TN>(c.b[e], ry, (unsigned)((k + e) * L + n0 + TN * lr) * 4u);
        if constexpr (ROWS) {
#pragma unroll
            for (int i = 0; i < MT; ++i) load_n<4>(c.a[i], rx, (unsigned)((16 * i + lr) * L + k) * 4u);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) load_n<MT>(c.a[e], rx, (unsigned)((k + e) * S + MT * lr) * 4u);
        }
    };
    const int chunks = (L + 15) / 16;
    auto k_loop = [&](auto tl) {
        constexpr int TL = decltype(tl)::value;      // column tiles that exist
        auto multiply = [&](Chunk &c, int ch) {
            if constexpr (ROWS) {                    // k past the end of W's rows: the next row's elements
                const int k = 16 * ch + 4 * lk;      // (unconditional: a branch here, and the loads in flight cannot be counted)
#pragma unroll
                for (int i = 0; i < (ROWS ? MT : 4); ++i)
#pragma unroll
                    for (int e = 0; e < (ROWS ? 4 : MT); ++e) c.a[i][e] = k + e < L ? c.a[i][e] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int t = 0; t < TL; ++t)
                        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ROWS ? c.a[ROWS ? i : 0][ROWS ? e : 0] : c.a[ROWS ? 0 : e][ROWS ? 0 : i],
                                                                         c.b[e][t], acc[i][t], 0, 0, 0);
        };
        Chunk c0, c1;
        load(c0, w);
        __builtin_amdgcn_sched_barrier(0);                  // issued in the order the loop consumes them
        load(c1, w + NW);
        __builtin_amdgcn_sched_barrier(0);
        for (int ch = w; ch < chunks; ch += 2 * NW) {       // chunks past the end are all zeros
            // a load ahead of the last use of the registers it replaces goes to others, and the copies at the end of the
            // trip wait for it
            multiply(c0, ch);
            __builtin_amdgcn_sched_barrier(0);
            load(c0, ch + 2 * NW);
            __builtin_amdgcn_sched_barrier(0);
            multiply(c1, ch + NW);
            __builtin_amdgcn_sched_barrier(0);
            load(c1, ch + 3 * NW);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // orders 64 k + 1 are the rule (bias column): their last tile has a single column, in MFMA tile 0
    const int live = min(TN, L - n0);
    if (live == 1) k_loop(std::integral_constant<int, 1>{});
    else k_loop(std::integral_constant<int, TN>{});

    // ---- the parts of the other wavefronts: wavefront t < TN sums MFMA tile t, in wavefront order ----
    float z[MT * 4][MT];
    if (w < live) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) load_n<MT>(z[4 * i + v], rz, (unsigned)(row_of(i, v) * S + MT * lr) * 4u);
    }
#pragma unroll
    for (int t = 0; t < TN; ++t)
        if (t != w && t < live) {
            floatx4 *d = lds + ((t * (NW - 1) + (w < t ? w : w - 1)) * MT) * 64 + lane;
#pragma unroll
            for (int i = 0; i < MT; ++i) d[i * 64] = acc[i][t];
        }
    __syncthreads();
    floatx4 res[MT];
    if (w < live) {
        floatx4 own[MT], sum[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            own[i] = acc[i][0];
#pragma unroll
            for (int t = 1; t < TN; ++t)
                if (t == w) own[i] = acc[i][t];
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) sum[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        const floatx4 *s = lds + (w * (NW - 1) * MT) * 64 + lane;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww)
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const floatx4 v = ww == w ? own[i] : s[((ww < w ? ww : ww - 1) * MT + i) * 64];
                sum[i] += v;
            }
        // ---- second product: the sums are its operand as they are (k = row_of(i, v) of this lane's group) ----
#pragma unroll
        for (int i = 0; i < MT; ++i) res[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = row_of(i, v) < S ? sum[i][v] : 0.f;
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    res[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[4 * i + v][m], x, res[m], 0, 0, 0);
            }
    }
    __syncthreads();          // the parts have been read
    // res[m][v]: row MT (4 lk + v) + m of the small dimension, column n0 + TN lr + w of the other
    constexpr int PO = 16 * TN + 4, PS = 16 * MT + 1;
    float *o = reinterpret_cast<float *>(lds);
    if (w < live) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int sm = MT * (4 * lk + v) + m, c = TN * lr + w;
                o[ROWS ? sm * PO + c : c * PS + sm] = res[m][v];
            }
    }
    __syncthreads();
    const int cols = min(16 * TN, L - n0);
    const bool div = pr.rv != nullptr;
    if constexpr (ROWS) {
        for (int e = tid; e < S * 16 * TN; e += 64 * NW) {
            const int m = e / (16 * TN), c = e & (16 * TN - 1);
            if (c < cols) {
                float v = o[m * PO + c];
                if (div) v = v / (pr.rv[m] * pr.cv[n0 + c] + gamma);
                pr.out[(long)m * L + n0 + c] = v;
            }
        }
    } else {
        for (int e = tid; e < cols * 16 * MT; e += 64 * NW) {
            const int c = e / (16 * MT), m = e & (16 * MT - 1);
            if (m < S) {
                float v = o[c * PS + m];
                if (div) v = v / (pr.rv[n0 + c] * pr.cv[m] + gamma);
                pr.out[(long)(n0 + c) * S + m] = v;
            }
        }
    }
}

template <int TN, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void precond_kernel(const PrecTable tab)
{
    constexpr int kParts = TN * (NW - 1) * 4 * 64;                        // floatx4
    constexpr int kOut = (64 * (16 * TN + 4) + 3) / 4, kOutT = (16 * TN * 65 + 3) / 4;
    constexpr int kLds = kParts > kOut ? (kParts > kOutT ? kParts : kOutT) : (kOut > kOutT ? kOut : kOutT);
    __shared__ floatx4 lds[kLds];
    // Workgroup i runs on XCD i mod 8: the tiles of a layer, which share W and G, meet in one L2.  Layers in groups of eight,
    // tile by tile; the layers of the last group, of less than eight, are spread over all XCDs.
    const int blk = blockIdx.x, full = tab.count >> 3;
    int prob, tile;
    if (blk < tab.group_blk[full]) {
        int lo = 0, hi = full - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (blk >= tab.group_blk[mid]) lo = mid;
            else hi = mid - 1;
        }
        const int off = blk - tab.group_blk[lo];
        prob = 8 * lo + (off & 7);
        tile = off >> 3;
    } else {
        const int rest = tab.count & 7;
        int r = 0;
        while (r + 1 < rest && blk >= tab.rest_blk[r + 1]) ++r;
        prob = 8 * full + r;
        tile = blk - tab.rest_blk[r];
    }
    const PrecProb &pr = tab.p[prob];
    if (tile >= pr.tiles) return;
    switch (pr.var) {
        case 0: precond_tile<1, TN, NW, true>(pr, tile, tab.gamma, lds); break;
        case 1: precond_tile<2, TN, NW, true>(pr, tile, tab.gamma, lds); break;
        case 3: precond_tile<4, TN, NW, true>(pr, tile, tab.gamma, lds); break;
        case 4: precond_tile<1, TN, NW, false>(pr, tile, tab.gamma, lds); break;
        case 5: precond_tile<2, TN, NW, false>(pr, tile, tab.gamma, lds); break;
        default: precond_tile<4, TN, NW, false>(pr, tile, tab.gamma, lds); break;
    }
}

}  // namespace

// One launch replaces two dependent ones and the intermediate, at the same number of MFMAs, so every layer with a
// dimension of at most 64 (four accumulator tiles of a wavefront) takes it; 16384: the byte offsets of a matrix fit 31 bits.
bool precond_fused_takes(int dA, int dG)
{
    return tuning().use_precond_fused && std::min(dA, dG) <= 64 && std::max(dA, dG) <= 16384;
}

hipError_t precond_fused_launch(const PrecJob *jobs, int n, float gamma, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // the longest workgroups first
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    auto mt = [&](int i) {
        const int m = (std::min(jobs[i].dA, jobs[i].dG) + 15) / 16;
        return m > 2 ? 4 : m;
    };
    auto cost = [&](int i) { return (long)std::max(jobs[i].dA, jobs[i].dG) * mt(i); };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost(a) > cost(b); });
    // 64-wide tiles, or 32-wide ones with twice the wavefronts on a tile's depth where those would leave CUs idle (on
    // the ResNet-110 shape, 671 of the 64-wide, the call takes 31 us with these and 46 with the others)
    long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (std::max(jobs[i].dA, jobs[i].dG) + 63) / 64;
    const bool few = tiles < tuning().precond_wide_tiles;
    const int bn = few ? 32 : 64;
    for (int g0 = 0; g0 < n; g0 += kMaxPrec) {
        PrecTable tab{};
        tab.count = std::min(kMaxPrec, n - g0);
        tab.gamma = gamma;
        double flops = 0.0;
        for (int k = 0; k < tab.count; ++k) {
            const PrecJob &j = jobs[order[g0 + k]];
            PrecProb &p = tab.p[k];
            p.W = j.W; p.A = j.A; p.G = j.G; p.out = j.out; p.rv = j.rv; p.cv = j.cv; p.dA = j.dA; p.dG = j.dG;
            const bool rows = j.dG <= j.dA;
            p.tiles = ((rows ? j.dA : j.dG) + bn - 1) / bn;
            p.var = mt(order[g0 + k]) - 1 + (rows ? 0 : 4);
            flops += 2.0 * j.dA * j.dG * ((double)j.dA + j.dG);
        }
        int blocks = 0;
        const int full = tab.count / 8;
        for (int g = 0; g < full; ++g) {
            tab.group_blk[g] = blocks;
            int most = 0;
            for (int k = 8 * g; k < 8 * g + 8; ++k) most = std::max(most, tab.p[k].tiles);
            blocks += 8 * most;
        }
        tab.group_blk[full] = blocks;
        for (int k = 8 * full; k < tab.count; ++k) {
            tab.rest_blk[k - 8 * full] = blocks;
            blocks += tab.p[k].tiles;
        }
        if (few) {
            KFAC_LAUNCH(KFAC_K_GEMM, s, (precond_kernel<2, 8>), dim3(blocks), dim3(512), 0, tab);
        } else {
            KFAC_LAUNCH(KFAC_K_GEMM, s, (precond_kernel<4, 4>), dim3(blocks), dim3(256), 0, tab);
        }
        timing_work(flops, flops);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kfac
