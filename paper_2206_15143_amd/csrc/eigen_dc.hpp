// Symmetric eigen-decomposition of factors up to order 1280: Householder reduction to tridiagonal form, divide and conquer
// (J. J. M. Cuppen, Numer. Math. 36, 1981; deflation and the rational interpolation of the secular equation as in
// R.-C. Li, LAPACK Working Note 89), and the reflectors applied to the eigenvectors of the tridiagonal matrix.
//
// The block Jacobi iteration of eigen.hip costs twelve sweeps of n / 16 dependent rounds that each stream the matrix and
// its vectors; the reduction here is one chain of n columns inside ONE launch, everything after it a few dozen short
// launches, and the flops are a tenth.  The 220 decompositions of the ResNet-110 shape (orders 16 to 577): 34.9 -> 7.3 ms, of
// them 5.3 dc_tridiag (577 columns at 9 us; the load path of one CU and the latency of the reductions, in about equal
// parts), 1.2 the six levels of merges, 0.5 dc_back.  Error of Eq. 13's result against float64 at order 577: 1.1e-5 with
// Jacobi, 2.1e-6 here.
//   dc_init       the lower triangle mirrored into the working matrix, vectors cleared
//   dc_tridiag    a workgroup of 8 wavefronts per matrix (all matrices at once, each on a CU of its own)
//   dc_leaf       the tree of halved tridiagonal matrices ends at orders up to 16: two-sided Jacobi in LDS, fp64
//   per level     dc_deflate (a workgroup per merge), dc_secular (16 lanes per root), dc_vectors (the orthogonal matrix of
//                 the rank-one problem), dc_product (its product with the vectors so far, fp32 MFMA)
//   dc_tfactor    the triangular factors of 64 reflectors each
//   dc_back       a workgroup per 16 or 32 eigenvectors applies all reflectors, the vectors in LDS
// Everything about the rank-one problems (poles, roots, differences between them) is fp64: roots of nearly equal poles come
// out accurate enough that the vectors need no correction to be orthogonal (the deflation keeps poles 2^-26 of the norm
// apart, 2^-53 / 2^-26 is below the rounding of the vectors to fp32).  No order of the eigenvalues, and none is made
// up: a deflated pair keeps its place, so a diagonal matrix gives Q = I exactly.
#pragma once

#include "common.hpp"

namespace kfac {

// Largest order: the LDS of dc_tridiag.  One matrix alone is where one CU per matrix does worst against the Jacobi iteration,
// which spreads over the chip: order 257, 513, 769, 1025, 1153, 1280 in ms, here / Jacobi: 1.5 / 5.4, 4.4 / 13.0, 11.2 / 24.0,
// 22.4 / 37.6, 33 / 48, 46 / 53; 32 matrices at 1280: 63 / 218.  Orders 24 to 32 alone in a call: 0.20 to 0.24 / 0.20.
constexpr int kDcMaxN = 1280;
constexpr int kDcLeaf = 16;         // (leaves of 32: a sweep costs eight times as much, a level less gains 0.12 ms)
constexpr int kDcTab = 256;        // matrices per launch (a 12 KB kernel argument)
constexpr int kDcNodes = 64;       // merges of a level at most (half of the leaves: 1280 / 16 rounded up to a power of two)

struct DcRot { int p, q; float c, s; };

struct DcProb {
    const float *M;
    float *Q, *v;
    int *info;
    char *ws;
    int n;
    int first;                     // first block of this matrix in the launch
};

struct DcTable {
    int count, sweeps, step;
    int iters;                     // steps of the iteration for a root at most
    DcProb p[kDcTab];
};

__host__ __device__ inline int dc_ld(int n) { return (n + 3) / 4 * 4; }
__host__ __device__ inline int dc_levels(int n)
{
    int l = 0;
    while (((n + (1 << l) - 1) >> l) > kDcLeaf) ++l;
    return l;
}
// node t of depth l: rows lo .. hi - 1
__host__ __device__ inline void dc_node(int n, int l, int t, int &lo, int &hi)
{
    lo = 0;
    hi = n;
    for (int b = l - 1; b >= 0; --b) {
        const int mid = lo + (hi - lo) / 2;
        if ((t >> b) & 1) lo = mid;
        else hi = mid;
    }
}

// Workspace of a matrix.
struct DcWs {
    float *A, *V0, *V1, *U, *T, *tau;
    double *d, *e, *dk, *zk, *root, *rho;
    int *org, *row, *kept, *cnt, *nrot;
    DcRot *rot;
    size_t bytes;
    __host__ __device__ DcWs(char *base, int n)
    {
        size_t off = 0;
        auto take = [&](size_t b) {
            char *p = base + off;
            off += (b + 255) / 256 * 256;
            return p;
        };
        const int ld = dc_ld(n), blocks = (n + 63) / 64;
        const size_t mat = (size_t)n * ld * sizeof(float);
        A = (float *)take(mat);
        V0 = (float *)take(mat);
        V1 = (float *)take(mat);
        U = (float *)take(mat);
        T = (float *)take((size_t)blocks * 64 * 64 * sizeof(float));
        tau = (float *)take((size_t)blocks * 64 * sizeof(float));
        d = (double *)take(n * sizeof(double));
        e = (double *)take(n * sizeof(double));
        dk = (double *)take(n * sizeof(double));
        zk = (double *)take(n * sizeof(double));
        root = (double *)take(n * sizeof(double));
        rho = (double *)take(kDcNodes * sizeof(double));
        org = (int *)take(n * sizeof(int));
        row = (int *)take(n * sizeof(int));
        kept = (int *)take(n * sizeof(int));
        cnt = (int *)take(kDcNodes * sizeof(int));
        nrot = (int *)take(kDcNodes * sizeof(int));
        rot = (DcRot *)take(n * sizeof(DcRot));
        bytes = off;
    }
    __device__ __forceinline__ float *V(int step) const { return (step & 1) ? V1 : V0; }    // the vectors before merge `step`
};

__device__ __forceinline__ const DcProb &dc_locate(const DcTable &tab, int &local)
{
    int lo = 0, hi = tab.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int)blockIdx.x >= tab.p[mid].first) lo = mid;
        else hi = mid - 1;
    }
    local = blockIdx.x - tab.p[lo].first;
    return tab.p[lo];
}

// 32 x 32 tiles on and below the diagonal: A full from the lower triangle of M, V cleared
__global__ __launch_bounds__(256) void dc_init_kernel(const DcTable tab)
{
    __shared__ float t[32][33];
    int local;
    const DcProb &pr = dc_locate(tab, local);
    const DcWs ws(pr.ws, pr.n);
    const int n = pr.n, ld = dc_ld(n);
    int bi = (int)((sqrtf(8.0f * (float)local + 1.0f) - 1.0f) * 0.5f);
    while ((bi + 1) * (bi + 2) / 2 <= local) ++bi;
    while (bi * (bi + 1) / 2 > local) --bi;
    const int bj = local - bi * (bi + 1) / 2;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    if (local == 0 && threadIdx.x == 0) *pr.info = 0;
    if (n <= kDcLeaf) return;                 // dc_leaf reads M itself
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bi * 32 + ty + 8 * r, j = bj * 32 + tx;
        const float x = i < n && j <= i ? pr.M[(long)i * n + j] : 0.f;
        t[ty + 8 * r][tx] = x;
        if (i < n && j < ld && (j <= i || j >= n)) ws.A[(long)i * ld + j] = x;
        if (i < n && j < ld) { ws.V0[(long)i * ld + j] = 0.f; ws.V1[(long)i * ld + j] = 0.f; }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bj * 32 + ty + 8 * r, j = bi * 32 + tx;    // the mirror image
        if (i < n && j < ld && j > i) ws.A[(long)i * ld + j] = t[tx][ty + 8 * r];
        if (i < n && j < ld && bi != bj) { ws.V0[(long)i * ld + j] = 0.f; ws.V1[(long)i * ld + j] = 0.f; }
    }
}

// Sums over a wavefront on the VALU alone (DPP; a shuffle is an LDS round trip): along rows of 16 lanes, then across rows.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dc_dpp(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dc_dpp(double x)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, false));
}
template <class F>
__device__ __forceinline__ F dc_sum63(F x)                 // valid in lane 63
{
    x += dc_dpp<0x111, 0xf>(x);          // row_shr 1, 2, 4, 8
    x += dc_dpp<0x112, 0xf>(x);
    x += dc_dpp<0x114, 0xf>(x);
    x += dc_dpp<0x118, 0xf>(x);
    x += dc_dpp<0x142, 0xa>(x);          // lane 15 of a row to the next one
    x += dc_dpp<0x143, 0xc>(x);          // lane 31 to the upper half
    return x;
}
__device__ __forceinline__ double dc_row_sum(double x)     // over 16 lanes, the same bits in all of them
{
    x += dc_dpp<0x128, 0xf>(x);          // row_ror 8, 4, 2, 1
    x += dc_dpp<0x124, 0xf>(x);
    x += dc_dpp<0x122, 0xf>(x);
    x += dc_dpp<0x121, 0xf>(x);
    return x;
}

// ---- reduction to tridiagonal form -----------------------------------------------------------------------------
// Panels of NB columns: inside a panel the matrix in memory stays as it is, column j is corrected by the panel's vectors
// V and W (in LDS) as it is needed, and A v by them after the pass over memory; the rank-2 NB update of the trailing
// matrix closes the panel.  Per column one read of the trailing matrix (the load path of one CU) and five barriers with
// a reduction between most of them (latency), in about equal parts at order 577.  Thread i owns row i of every vector.
// Column j's reflector replaces row j of A (zeros up to its one).
constexpr int kTriWaves = 8;

// A barrier for what the wavefronts exchange through LDS: memory accesses under way stay under way (the one behind
// __syncthreads waits for the store of the reflector and for the row fetched ahead).
__device__ __forceinline__ void dc_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kTriLds = (2 * 16 * (768 + 16) + kTriWaves * (768 + 16)) * 4;

// R rows of 256 LC columns per wavefront and step, two steps under way
template <int CH, int NB, int R>
__device__ __forceinline__ void dc_tridiag(const DcProb &pr, float *lds)
{
    constexpr int NW = kTriWaves, NT = 64 * NW;
    constexpr int NM = 256 * CH, NP = NM + 16, RP = (NP + NT - 1) / NT;
    static_assert((2 * NB + NW) * NP * 4 <= kTriLds, "LDS of the kernel");
    __shared__ double part[2][16];
    __shared__ float pq[2 * 16];
    __shared__ float alpha_s;
    const DcWs ws(pr.ws, pr.n);
    const int n = pr.n, ld = dc_ld(n);
    float *A = ws.A;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(A, 0, n * ld * 4, 0x00020000);
    float *V = lds, *W = lds + NB * NP, *red = lds + 2 * NB * NP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < 2 * NB * NP; e += NT) lds[e] = 0.f;
    if (tid < 32) part[tid >> 4][tid & 15] = 0.0;
    __syncthreads();
    for (int p0 = 0; p0 < n - 2; p0 += NB) {
        const int nbk = min(NB, n - 2 - p0);
        float next[RP];                                  // row j as the panel began, fetched a column ahead
        auto fetch = [&](int j) {
#pragma unroll
            for (int q = 0; q < RP; ++q) next[q] = A[(long)j * ld + min(tid + NT * q, n - 1)];
        };
        fetch(p0);
        int least = n;                                   // of the first rows of the panel's passes: n if there was none
        for (int k = 0; k < nbk; ++k) {
            const int j = p0 + k;
            // ---- column j (= row j), corrected; its norm below the subdiagonal ----
            float a[RP];
            double ss = 0.0;
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int i = tid + NT * q;
                a[q] = i >= j && i < n ? next[q] : 0.f;
            }
            if (k + 1 < nbk) fetch(j + 1);
#pragma unroll 4
            for (int l = 0; l < k; ++l) {
                const float wj = W[l * NP + j], vj = V[l * NP + j];
#pragma unroll
                for (int q = 0; q < RP; ++q) {
                    const int i = min(tid + NT * q, NP - 1);
                    a[q] = __builtin_fmaf(-V[l * NP + i], wj, a[q]);
                    a[q] = __builtin_fmaf(-W[l * NP + i], vj, a[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int i = tid + NT * q;
                if (i >= n) a[q] = 0.f;
                if (i == j) ws.d[j] = a[q];
                if (i == j + 1) alpha_s = a[q];
                if (i >= j + 2) ss += (double)a[q] * (double)a[q];
            }
            ss = dc_sum63(ss);
            if (lane == 63) part[0][w] = ss;
            dc_lds_barrier();
            const double xn2 = dc_row_sum(part[0][lane & 15]);
            // A column with nothing below the subdiagonal (tau = 0, W = 0) passes over no rows: a diagonal matrix of order 1153
            // takes 4.8 instead of 32 ms.  Up to order 256 the passes are short and the test costs as much (1.7 % at order 145,
            // 0.5 % above).
            const int i0 = CH > 1 ? __builtin_amdgcn_readfirstlane(xn2 == 0.0 ? n : j + 1 + w) : j + 1 + w;
            least = min(least, i0);
            const double alpha = alpha_s;
            double beta = alpha, tau = 0.0, scale = 0.0;
            if (xn2 > 0.0) {
                // beta = -sign(alpha) r, tau = (beta - alpha) / beta, v = x / (alpha - beta); the hardware's reciprocal
                // (square root) and two steps of Newton's iteration
                const double r2 = alpha * alpha + xn2;
                double ir = __builtin_amdgcn_rsq(r2);
                ir = ir * (1.5 - 0.5 * r2 * ir * ir);
                ir = ir * (1.5 - 0.5 * r2 * ir * ir);
                const double r = r2 * ir, den = fabs(alpha) + r;
                double id = __builtin_amdgcn_rcp(den);
                id = id * (2.0 - den * id);
                id = id * (2.0 - den * id);
                beta = alpha > 0.0 ? -r : r;
                tau = 1.0 + fabs(alpha) * ir;
                scale = alpha > 0.0 ? id : -id;
            }
            const float tauf = (float)tau;
            float v[RP];
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int i = tid + NT * q;
                // the product in fp64: the reciprocal of a column's norm need not be in the range of fp32 (rows of a feature that
                // no longer fires decay to a few multiples of 2^-149)
                v[q] = i <= j || i >= n ? 0.f : (i == j + 1 ? 1.f : (float)((double)a[q] * scale));
                if (i < NP) V[k * NP + i] = v[q];
            }
            dc_lds_barrier();
            // ---- A v over the trailing matrix: rows j + 1 + w, + NW, ..., lanes along the columns; beside the first
            // loads W_l^T v and V_l^T v, a wavefront per l ----
            const float *vk = V + k * NP;
            const int c0 = (j + 1) & ~3;
            floatx4 acc[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
            auto dots = [&] {
                for (int l = w; l < k; l += NW) {
                    float sp = 0.f, sq = 0.f;
#pragma unroll 4
                    for (int i = (j + 1 & ~63) + lane; i < n; i += 64) {        // (v is zero up to j)
                        sp = __builtin_fmaf(W[l * NP + i], vk[i], sp);
                        sq = __builtin_fmaf(V[l * NP + i], vk[i], sq);
                    }
                    sp = dc_sum63(sp);
                    sq = dc_sum63(sq);
                    if (lane == 63) { pq[2 * l] = sp; pq[2 * l + 1] = sq; }
                }
            };
            auto rows = [&](auto live) {
                constexpr int LC = decltype(live)::value;       // chunks of 256 columns that exist
                typedef int dint4 __attribute__((ext_vector_type(4)));
                dint4 x0[R][LC], x1[R][LC];
                unsigned vo[LC];
#pragma unroll
                for (int c = 0; c < LC; ++c) {
                    const int col = c0 + 256 * c + 4 * lane;
                    vo[c] = col < ld ? 4u * (unsigned)col : 0x80000000u;     // outside the buffer: zeros, no traffic
                }
                auto load = [&](dint4 (&x)[R][LC], int i) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int row = i + NW * r;
                        const unsigned so = row < n ? (unsigned)(row * ld) * 4u : 0x7fffff00u;
#pragma unroll
                        for (int c = 0; c < LC; ++c)
                            x[r][c] = __builtin_bit_cast(dint4, __builtin_amdgcn_raw_buffer_load_b128(ra, vo[c] + so, 0, 0));
                    }
                };
                auto add = [&](const dint4 (&x)[R][LC], int i) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float xi = vk[min(i + NW * r, NP - 1)];       // (zero from n on)
#pragma unroll
                        for (int c = 0; c < LC; ++c)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[c][e] = __builtin_fmaf(__int_as_float(x[r][c][e]), xi, acc[c][e]);
                    }
                };
                load(x0, i0);
                __builtin_amdgcn_sched_barrier(0);
                load(x1, i0 + NW * R);
                __builtin_amdgcn_sched_barrier(0);
                dots();
                __builtin_amdgcn_sched_barrier(0);
                for (int i = i0; i < n; i += 2 * NW * R) {
                    add(x0, i);
                    __builtin_amdgcn_sched_barrier(0);
                    load(x0, i + 2 * NW * R);
                    __builtin_amdgcn_sched_barrier(0);
                    add(x1, i + NW * R);
                    __builtin_amdgcn_sched_barrier(0);
                    load(x1, i + 3 * NW * R);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            const int chunks = (n - c0 + 255) / 256;
            if (CH >= 5 && chunks == 5) rows(std::integral_constant<int, CH < 5 ? CH : 5>{});
            else if (CH >= 5 && chunks == 4) rows(std::integral_constant<int, CH < 4 ? CH : 4>{});
            else if (CH >= 3 && chunks == 3) rows(std::integral_constant<int, CH < 3 ? CH : 3>{});
            else if (CH >= 2 && chunks == 2) rows(std::integral_constant<int, CH < 2 ? CH : 2>{});
            else rows(std::integral_constant<int, 1>{});
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int col = c0 + 256 * c + 4 * lane;
                if (col < n) *reinterpret_cast<floatx4 *>(red + w * NP + col) = acc[c];
            }
            dc_lds_barrier();
            // the reflector, behind the loads (a load is not seen before the stores ahead of it have been acknowledged)
#pragma unroll
            for (int q = 0; q < RP; ++q)
                if (tid + NT * q < ld) A[(long)j * ld + tid + NT * q] = v[q];
            if (tid == 0) { ws.e[j] = beta; ws.tau[j] = tauf; }
            float y[RP];
            double dot = 0.0;
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int i = tid + NT * q;
                y[q] = 0.f;
                if (i > j && i < n) {
#pragma unroll
                    for (int s = 0; s < NW; ++s) y[q] += red[s * NP + i];
#pragma unroll 4
                    for (int l = 0; l < k; ++l) {
                        y[q] = __builtin_fmaf(-V[l * NP + i], pq[2 * l], y[q]);
                        y[q] = __builtin_fmaf(-W[l * NP + i], pq[2 * l + 1], y[q]);
                    }
                    dot += (double)y[q] * (double)v[q];
                }
            }
            dot = dc_sum63(dot);
            if (lane == 63) part[1][w] = dot;
            dc_lds_barrier();
            const double all = dc_row_sum(part[1][lane & 15]);
            const float half = (float)(0.5 * tau * all);
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int i = tid + NT * q;
                if (i < NP) W[k * NP + i] = tauf * __builtin_fmaf(-half, v[q], y[q]);
            }
            dc_lds_barrier();
        }
        for (int e = tid; e < (NB - nbk) * NP; e += NT) { V[nbk * NP + e] = 0.f; W[nbk * NP + e] = 0.f; }
        __syncthreads();
        // ---- A -= V W^T + W V^T from row and column p1 on: 16 x 16 tiles of the lower triangle, each stored twice.
        // An MFMA result column is a matrix row here, so that a lane's four values are neighbours of a row. ----
        const int p1 = p0 + nbk, nt = (n - p1 + 15) / 16;
        const int lr = lane & 15, lk = lane >> 4;
        const bool al = (p1 & 3) == 0;
        // a wavefront takes tile rows w, w + NW, ..., the lengths of two of them added up even out; none if all W are zero
        for (int ti = least == n ? nt : w; ti < nt; ti += NW)
            for (int t0 = 0; t0 <= ti; t0 += 4) {
                const int ri = p1 + 16 * ti, i = ri + lr;
                float *row = A + (long)min(i, n - 1) * ld;
                floatx4 old[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = p1 + 16 * (t0 + u) + 4 * lk;
                    const bool whole = al && c + 3 < ld;
                    if (t0 + u > ti) continue;
                    if (whole) old[u] = *reinterpret_cast<const floatx4 *>(row + c);
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) old[u][e] = c + e < n ? row[c + e] : 0.f;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (t0 + u > ti) break;
                    const int cj = p1 + 16 * (t0 + u), c = cj + 4 * lk;
                    const bool whole = al && c + 3 < ld;
                    floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < NB / 4; ++q) {
                        const int l = (4 * q + lk) * NP;
                        s = __builtin_amdgcn_mfma_f32_16x16x4f32(W[l + cj + lr], V[l + ri + lr], s, 0, 0, 0);
                        s = __builtin_amdgcn_mfma_f32_16x16x4f32(V[l + cj + lr], W[l + ri + lr], s, 0, 0, 0);
                    }
                    s = old[u] - s;
                    if (i < n) {
                        if (whole) *reinterpret_cast<floatx4 *>(row + c) = s;
                        else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (c + e < n) row[c + e] = s[e];
                        }
                        if (t0 + u != ti) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (c + e < n) A[(long)(c + e) * ld + i] = s[e];
                        }
                    }
                }
            }
        __syncthreads();
    }
    if (tid == 0) {
        ws.d[n - 2] = A[(long)(n - 2) * ld + n - 2];
        ws.e[n - 2] = A[(long)(n - 2) * ld + n - 1];
        ws.d[n - 1] = A[(long)(n - 1) * ld + n - 1];
    }
    for (int j = n - 2 + tid; j < (n + 63) / 64 * 64; j += NT) ws.tau[j] = 0.f;     // no reflectors from n - 2 on
}

__global__ __launch_bounds__(64 * kTriWaves, 1) void dc_tridiag_kernel(const DcTable tab)
{
    __shared__ __attribute__((aligned(16))) float lds[kTriLds / 4];
    const DcProb &pr = tab.p[blockIdx.x];
    if (pr.n <= kDcLeaf) return;
    if (pr.n <= 256) dc_tridiag<1, 16, 8>(pr, lds);
    else if (pr.n <= 768) dc_tridiag<3, 16, 4>(pr, lds);
    else dc_tridiag<5, 8, 3>(pr, lds);
}

// ---- leaves ------------------------------------------------------------------------------------------------------
// Pair k of round r of a round-robin tournament over m (even) players.
__device__ __forceinline__ void dc_pair(int m, int r, int k, int &a, int &b)
{
    if (k == 0) { a = m - 1; b = r; }
    else { a = (r + k) % (m - 1); b = (r - k + (m - 1)) % (m - 1); }
    if (a > b) { const int t = a; a = b; b = t; }
}

// Cyclic two-sided Jacobi of one leaf (or of a whole matrix up to order 16) in LDS, one wavefront, 8 disjoint rotations
// at a time.
__global__ __launch_bounds__(64) void dc_leaf_kernel(const DcTable tab)
{
    constexpr int N = kDcLeaf;
    __shared__ double S[N][N + 1], R[N][N + 1];
    int local;
    const DcProb &pr = dc_locate(tab, local);
    const DcWs ws(pr.ws, pr.n);
    const int n = pr.n, L = dc_levels(n), tid = threadIdx.x;
    int lo, hi;
    dc_node(n, L, local, lo, hi);
    const int s = hi - lo;
    double most = 0.0;
    for (int e = tid; e < N * N; e += 64) {
        const int i = e / N, j = e - i * N;
        double x = 0.0;
        if (i < s && j < s) {
            if (L == 0) {
                x = pr.M[max(i, j) * n + min(i, j)];
            } else if (i == j) {
                x = ws.d[lo + i];
                if (i == 0 && lo > 0) x -= fabs(ws.e[lo - 1]);           // the cuts above and below take |e| each
                if (i == s - 1 && hi < n) x -= fabs(ws.e[hi - 1]);
            } else if (i == j + 1 || j == i + 1) {
                x = ws.e[lo + min(i, j)];
            }
        }
        S[i][j] = x;
        R[i][j] = i == j ? 1.0 : 0.0;
        most = fmax(most, fabs(x));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = fmax(most, __shfl_xor(most, o));
    __syncthreads();
    const double tol = 1e-11 * most;
    const int pk = tid & 7, part = tid >> 3;           // rotation, and which two elements of its rows and columns
    bool open = true;
    for (int sw = 0; sw < tab.sweeps && open; ++sw) {
        bool any = false;
        for (int rd = 0; rd < N - 1; ++rd) {
            int p, q;
            dc_pair(N, rd, pk, p, q);
            const double app = S[p][p], aqq = S[q][q], apq = S[p][q];
            double cs = 1.0, sn = 0.0;
            if (fabs(apq) > tol) {
                const double th = (aqq - app) / (2.0 * apq);
                const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(1.0 + th * th));
                cs = 1.0 / sqrt(1.0 + t * t);
                sn = t * cs;
                any = true;
            }
            __syncthreads();
            {
                double sp[2], sq[2], rp[2], rq[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * part + e;
                    sp[e] = S[i][p]; sq[e] = S[i][q]; rp[e] = R[i][p]; rq[e] = R[i][q];
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * part + e;
                    S[i][p] = cs * sp[e] - sn * sq[e];
                    S[i][q] = sn * sp[e] + cs * sq[e];
                    R[i][p] = cs * rp[e] - sn * rq[e];
                    R[i][q] = sn * rp[e] + cs * rq[e];
                }
            }
            __syncthreads();
            {
                double sp[2], sq[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) { sp[e] = S[p][2 * part + e]; sq[e] = S[q][2 * part + e]; }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    S[p][2 * part + e] = cs * sp[e] - sn * sq[e];
                    S[q][2 * part + e] = sn * sp[e] + cs * sq[e];
                }
            }
            __syncthreads();
        }
        open = __syncthreads_or(any ? 1 : 0) != 0;
    }
    if (open && tid == 0) *pr.info = 1;                 // the budget ended on a sweep that still rotated
    const int ld = dc_ld(n);
    for (int e = tid; e < N * N; e += 64) {
        const int k = e / N, i = e - k * N;             // eigenvector k
        if (k >= s || i >= s) continue;
        if (L == 0) pr.Q[i * n + k] = (float)R[i][k];
        else ws.V0[(long)(lo + k) * ld + lo + i] = (float)R[i][k];
    }
    if (tid < s) {
        if (L == 0) pr.v[tid] = (float)S[tid][tid];
        else ws.d[lo + tid] = S[tid][tid];
    }
}

// ---- one merge: D + rho z z^T ------------------------------------------------------------------------------------
// Merge step `tab.step` of every matrix: depth levels - 1 - step.  False when the matrix is complete.
__device__ __forceinline__ bool dc_merge(const DcProb &pr, int step, int local, int per, int &node, int &sub, int &lo, int &mid, int &hi)
{
    const int l = dc_levels(pr.n) - 1 - step;
    if (l < 0) return false;
    node = local / per;
    sub = local - node * per;
    dc_node(pr.n, l, node, lo, hi);
    mid = lo + (hi - lo) / 2;
    return true;
}

// Poles sorted, those that do not take part (tiny z) or coincide with their neighbour (rotated apart) set aside.
// LDS: order of a merge at most kDcMaxN.
__global__ __launch_bounds__(256) void dc_deflate_kernel(const DcTable tab)
{
    __shared__ double dd[kDcMaxN], zz[kDcMaxN], kd[kDcMaxN], kz[kDcMaxN];
    __shared__ short si[kDcMaxN], ki[kDcMaxN];
    __shared__ double sh[4];
    __shared__ unsigned long long close[kDcMaxN / 64 + 4];
    __shared__ int base, waves[4], rots;
    int local, node, sub, lo, mid, hi;
    const DcProb &pr = dc_locate(tab, local);
    if (!dc_merge(pr, tab.step, local, 1, node, sub, lo, mid, hi)) return;
    const DcWs ws(pr.ws, pr.n);
    const int ld = dc_ld(pr.n), s = hi - lo, n1 = mid - lo, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float *V = ws.V(tab.step);
    const double e = ws.e[mid - 1];
    const double sg = e < 0.0 ? -1.0 : 1.0;
    double z2 = 0.0, most = 0.0;
    for (int j = tid; j < s; j += 256) {
        double x = ws.d[lo + j];
        if (!(fabs(x) < 1e300)) x = 1e300;                        // a total order whatever the input held
        const double z = j < n1 ? V[(long)(lo + j) * ld + mid - 1] : sg * V[(long)(lo + j) * ld + mid];
        dd[j] = x;
        zz[j] = z;
        kd[j] = 0.0; kz[j] = 0.0; ki[j] = 0;
        z2 += z * z;
        most = fmax(most, fabs(x));
    }
    z2 = dc_sum63(z2);
    if (lane == 63) sh[w] = z2;
    __syncthreads();
    z2 = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = fmax(most, __shfl_xor(most, o));
    if (lane == 0) sh[w] = most;
    if (tid == 0) { base = 0; rots = 0; }
    __syncthreads();
    most = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    const double zn = z2 > 0.0 ? 1.0 / sqrt(z2) : 0.0;
    const double rho = fabs(e) * z2;
    const double tol = fmax(most, rho) * 1.4901161193847656e-8;   // 2^-26
    // rank of every pole: the place of row j in increasing order
    for (int j = tid; j < s; j += 256) {
        const double x = dd[j];
        int r = 0;
        for (int i = 0; i < s; ++i) r += dd[i] < x || (dd[i] == x && i < j);
        si[r] = (short)j;
    }
    __syncthreads();
    // those that take part, in order
    for (int r0 = 0; r0 < s; r0 += 256) {
        const int r = r0 + tid;
        const int j = r < s ? si[r] : 0;
        const bool keep = r < s && rho * fabs(zz[j] * zn) > tol;
        const unsigned long long m = __ballot(keep);
        if (lane == 0) waves[w] = __popcll(m);
        __syncthreads();
        int at = base + __popcll(m & ((1ull << lane) - 1));
        for (int q = 0; q < w; ++q) at += waves[q];
        if (keep) { kd[at] = dd[j]; kz[at] = zz[j] * zn; ki[at] = (short)j; }
        if (r < s) ws.kept[lo + j] = -1;
        __syncthreads();
        if (tid == 0) base += waves[0] + waves[1] + waves[2] + waves[3];
        __syncthreads();
    }
    int k = base;
    // Neighbours so close that a rotation may clear one of the two z.  The survivor of a pair meets the next pole whether or
    // not those two were close before; everything else in the chain is left alone.
    auto meet = [&](int p, int q) {
        const double h = kz[p] * kz[p] + kz[q] * kz[q];
        return (kd[q] - kd[p]) * fabs(kz[p] * kz[q]) <= tol * h;
    };
    bool any = false;
    for (int r0 = 0; r0 < k; r0 += 256) {
        const int r = r0 + tid;
        const bool c = r + 1 < k && meet(r, r + 1);
        const unsigned long long m = __ballot(c);
        if (lane == 0) close[r0 / 64 + w] = m;
        any |= c;
    }
    if (__syncthreads_or(any ? 1 : 0)) {
        if (tid == 0) {
            int nr = 0, done = 0;
            const int words = (k + 63) / 64;
            for (int wd = 0; wd < words; ++wd) {
                unsigned long long m = close[wd];
                while (m) {
                    const int r = 64 * wd + __ffsll(m) - 1;
                    m &= m - 1;
                    if (r < done) continue;             // settled with the chain before it
                    int p = r;
                    while (p + 1 < k && meet(p, p + 1)) {
                        const int q = p + 1;
                        const double h = sqrt(kz[p] * kz[p] + kz[q] * kz[q]);
                        const double c = kz[q] / h, sn = -kz[p] / h, a = kd[p], b = kd[q];
                        kz[q] = h;
                        ws.d[lo + ki[p]] = a * c * c + b * sn * sn;
                        kd[q] = a * sn * sn + b * c * c;
                        ws.rot[lo + nr++] = DcRot{ki[p], ki[q], (float)c, (float)sn};
                        kz[p] = 0.0;                   // gone
                        p = q;
                    }
                    done = p;
                }
            }
            rots = nr;
            base = 0;
        }
        __syncthreads();
        // close the gaps (every thread reads its elements before any is written)
        for (int r0 = 0; r0 < k; r0 += 256) {
            const int r = r0 + tid;
            const bool keep = r < k && kz[r] != 0.0;
            const double a = r < k ? kd[r] : 0.0, b = r < k ? kz[r] : 0.0;
            const short i = r < k ? ki[r] : 0;
            const unsigned long long m = __ballot(keep);
            if (lane == 0) waves[w] = __popcll(m);
            __syncthreads();
            int at = base + __popcll(m & ((1ull << lane) - 1));
            for (int q = 0; q < w; ++q) at += waves[q];
            if (keep) { kd[at] = a; kz[at] = b; ki[at] = i; }
            __syncthreads();
            if (tid == 0) base += waves[0] + waves[1] + waves[2] + waves[3];
            __syncthreads();
        }
        k = base;
    }
    for (int r = tid; r < k; r += 256) {
        ws.dk[lo + r] = kd[r];
        ws.zk[lo + r] = kz[r];
        ws.row[lo + r] = ki[r];
        ws.kept[lo + ki[r]] = r;
    }
    if (tid == 0) { ws.cnt[node] = k; ws.nrot[node] = rots; ws.rho[node] = rho; }
}

// Root i of 1 / rho + sum_j z_j^2 / (d_j - x) between d_i and d_{i+1} (the last one up to d_i + rho), as a distance from
// the nearer pole.  Sixteen lanes sum; each side of the root is replaced by a constant and its nearest pole with the
// same value and slope, the zero of that is the next iterate, and a bracket guards it.  info = 1 if the step budget ran out.
__global__ __launch_bounds__(256) void dc_secular_kernel(const DcTable tab)
{
    int local, node, sub, lo, mid, hi;
    const DcProb &pr = dc_locate(tab, local);
    const int l = dc_levels(pr.n) - 1 - tab.step;
    if (l < 0) return;
    const int most = (pr.n + (1 << l) - 1) >> l;
    dc_merge(pr, tab.step, local, (most + 15) / 16, node, sub, lo, mid, hi);
    const DcWs ws(pr.ws, pr.n);
    const int k = ws.cnt[node], lane = threadIdx.x & 15;
    const int i = min(sub * 16 + (int)(threadIdx.x >> 4), k - 1);      // surplus groups repeat the last root
    if (k <= 0) return;
    const double *d = ws.dk + lo, *z = ws.zk + lo;
    const double rho = ws.rho[node], ri = 1.0 / rho;
    const bool last = i == k - 1;
    const double gap = last ? rho : d[i + 1] - d[i];
    double psi, dpsi, phi, dphi;
    int org = i;
    double dorg = d[i];
    auto eval = [&](double x) {
        psi = dpsi = phi = dphi = 0.0;
        for (int j = lane; j < k; j += 16) {
            const double q = z[j] / ((d[j] - dorg) - x), t = z[j] * q;
            if (j <= i) { psi += t; dpsi += q * q; }
            else { phi += t; dphi += q * q; }
        }
        psi = dc_row_sum(psi);
        dpsi = dc_row_sum(dpsi);
        phi = dc_row_sum(phi);
        dphi = dc_row_sum(dphi);
    };
    double a = 0.0, b = gap, xl = 0.0, xr = last ? 1.01 * gap : gap;   // poles of the interpolation, bracket
    double x = 0.5 * gap;
    eval(x);
    if (!last && ri + psi + phi < 0.0) {                               // the root is nearer to the upper pole
        org = i + 1;
        dorg = d[i + 1];
        a = -gap;
        b = 0.0;
        xl = -0.5 * gap;
        xr = 0.0;
        x = -0.5 * gap;
    } else if (!last) {
        xr = 0.5 * gap;
    }
    for (int it = 0;; ++it) {
        const double f = ri + psi + phi;
        if (f < 0.0) xl = fmax(xl, x);
        else xr = fmin(xr, x);
        if (fabs(f) <= 8e-16 * (ri + fabs(psi) + phi) || !(xr - xl > 2e-16 * fmax(fabs(xl), fabs(xr)))) break;
        if (it == tab.iters) {
            if (lane == 0) *pr.info = 1;
            break;
        }
        const double da = a - x, db = b - x;
        const double s1 = da * da * dpsi;
        double nx;
        if (last) {
            const double c = ri + psi - da * dpsi;
            nx = a + s1 / c;
        } else {
            const double s2 = db * db * dphi;
            const double c = ri + (psi - da * dpsi) + (phi - db * dphi);
            // c (a - x)(b - x) + s1 (b - x) + s2 (a - x) = 0, one of a and b is 0
            const double B = c * (a + b) + s1 + s2, C = s1 * b + s2 * a;
            const double disc = B * B - 4.0 * c * C;
            const double root = sqrt(fmax(disc, 0.0));
            const double q = 0.5 * (B + (B >= 0.0 ? root : -root));
            const double x1 = C / q, x2 = q / c;
            nx = x1 > xl && x1 < xr ? x1 : x2;
        }
        if (!(nx > xl && nx < xr)) nx = 0.5 * (xl + xr);
        if (fabs(nx - x) <= 2e-16 * fabs(nx)) break;
        x = nx;
        eval(x);
    }
    if (lane == 0 && sub * 16 + (int)(threadIdx.x >> 4) < k) {
        ws.root[lo + i] = x;
        ws.org[lo + i] = org;
    }
}

// The orthogonal matrix of the merge, rows = old vectors, columns = new ones: z_r / (d_r - x_c), scaled; a row or column
// set aside is a row or column of the identity.  64 columns per workgroup.  Leaves the new eigenvalues in d.
__global__ __launch_bounds__(256) void dc_vectors_kernel(const DcTable tab)
{
    __shared__ double pd[kDcMaxN], pz[kDcMaxN];
    __shared__ double part[4][64];
    int local, node, sub, lo, mid, hi;
    const DcProb &pr = dc_locate(tab, local);
    const int l = dc_levels(pr.n) - 1 - tab.step;
    if (l < 0) return;
    const int most = (pr.n + (1 << l) - 1) >> l;
    dc_merge(pr, tab.step, local, (most + 63) / 64, node, sub, lo, mid, hi);
    const DcWs ws(pr.ws, pr.n);
    const int s = hi - lo, ld = dc_ld(pr.n), tid = threadIdx.x, cl = tid & 63, g = tid >> 6;
    if (sub * 64 >= s) return;
    for (int r = tid; r < s; r += 256) {
        const int kp = ws.kept[lo + r];
        pd[r] = kp >= 0 ? ws.dk[lo + kp] : 0.0;
        pz[r] = kp >= 0 ? ws.zk[lo + kp] : 0.0;
    }
    __syncthreads();
    const int c = sub * 64 + cl;
    const int kc = c < s ? ws.kept[lo + c] : -1;
    const double dorg = kc >= 0 ? ws.dk[lo + ws.org[lo + kc]] : 0.0, x = kc >= 0 ? ws.root[lo + kc] : 0.0;
    double nn = 0.0;
    if (kc >= 0)
        for (int r = g; r < s; r += 4) {
            const double q = pz[r] / ((pd[r] - dorg) - x);
            if (pz[r] != 0.0) nn += q * q;
        }
    part[g][cl] = nn;
    __syncthreads();
    nn = (part[0][cl] + part[1][cl]) + (part[2][cl] + part[3][cl]);
    const double sc = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    if (c < s) {
        for (int r = g; r < s; r += 4) {
            double u;
            if (kc < 0) u = r == c ? 1.0 : 0.0;
            else u = pz[r] != 0.0 ? pz[r] / ((pd[r] - dorg) - x) * sc : 0.0;
            ws.U[(long)(lo + r) * ld + lo + c] = (float)u;
        }
        if (g == 0 && kc >= 0) ws.d[lo + c] = dorg + x;
    }
    const int nrot = ws.nrot[node];
    if (nrot == 0) return;
    __syncthreads();                                  // this workgroup's columns are complete
    if (g == 0 && c < s)
        for (int t = nrot - 1; t >= 0; --t) {         // the rotations of the old vectors, the last one first
            const DcRot rt = ws.rot[lo + t];
            float *up = ws.U + (long)(lo + rt.p) * ld + lo + c, *uq = ws.U + (long)(lo + rt.q) * ld + lo + c;
            const float a = *up, b = *uq;
            *up = rt.c * a - rt.s * b;
            *uq = rt.s * a + rt.c * b;
        }
}

// New vectors: V' = U^T V on the merge's block, 64 x 64 tiles, the wavefronts split K (see precond.hip for the operand
// layout).  The old vectors are block diagonal: the columns of one half have their rows in that half alone.
__global__ __launch_bounds__(256, 2) void dc_product_kernel(const DcTable tab)
{
    __shared__ floatx4 lds[4 * 3 * 4 * 64];
    int local, node, sub, lo, mid, hi;
    const DcProb &pr = dc_locate(tab, local);
    const int l = dc_levels(pr.n) - 1 - tab.step;
    if (l < 0) return;
    const int side = ((((pr.n + (1 << l) - 1) >> l)) + 63) / 64;
    dc_merge(pr, tab.step, local, side * side, node, sub, lo, mid, hi);
    const DcWs ws(pr.ws, pr.n);
    const int ld = dc_ld(pr.n), s = hi - lo;
    const int m0 = sub / side * 64, n0 = sub % side * 64;
    if (m0 >= s || n0 >= s) return;
    const int n1 = mid - lo;
    const int kb = n0 >= n1 ? n1 : 0, ke = n0 + 64 <= n1 ? n1 : s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    // loads run up to three columns past the matrix: rows are 4 floats apart at least, the buffers' ends are checked
    const long bytes = (long)pr.n * ld * 4;
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(ws.U, 0, (int)bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(ws.V(tab.step)), 0, (int)bytes, 0x00020000);
    typedef int dint4 __attribute__((ext_vector_type(4)));
    auto ld4 = [&](__amdgpu_buffer_rsrc_t r, unsigned off) {
        const dint4 v = __builtin_bit_cast(dint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        return floatx4{__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3])};
    };
    floatx4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    const unsigned uo = (unsigned)(lo + m0 + 4 * lr) * 4u, vo = (unsigned)(lo + n0 + 4 * lr) * 4u;
    auto load = [&](floatx4 (&a)[4], floatx4 (&b)[4], int k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int kk = k + 4 * e + lk;
            const unsigned r = kk < ke ? (unsigned)((lo + kk) * ld) * 4u : 0x80000000u;   // past the range: zeros
            a[e] = ld4(ru, r + uo);
            b[e] = ld4(rv, r + vo);
        }
    };
    auto multiply = [&](const floatx4 (&a)[4], const floatx4 (&b)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e][i], b[e][t], acc[i][t], 0, 0, 0);
    };
    floatx4 a0[4], b0[4], a1[4], b1[4];
    load(a0, b0, kb + 16 * w);
    __builtin_amdgcn_sched_barrier(0);
    load(a1, b1, kb + 16 * w + 64);
    __builtin_amdgcn_sched_barrier(0);
    for (int k = kb + 16 * w; k < ke; k += 128) {
        multiply(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        load(a0, b0, k + 128);
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        load(a1, b1, k + 192);
        __builtin_amdgcn_sched_barrier(0);
    }
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
    float *o = reinterpret_cast<float *>(lds);          // 64 rows of 68: row 4 (4 lk + v) + i, column 4 lr + w
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[(4 * (4 * lk + v) + i) * 68 + 4 * lr + w] = sum[i][v];
    __syncthreads();
    float *dst = ws.V(tab.step + 1);
    for (int e = tid; e < 64 * 64; e += 256) {
        const int m = e >> 6, c = e & 63;
        if (m0 + m < s && n0 + c < s) dst[(long)(lo + m0 + m) * ld + lo + n0 + c] = o[m * 68 + c];
    }
}

// ---- the reflectors ------------------------------------------------------------------------------------------------
// T of 64 reflectors, H_0 H_1 ... = I - Y T Y^T with the reflectors in the columns of Y (the rows of A): their Gram matrix
// on the MFMA units, then column by column T[0:i, i] = -tau_i T[0:i, 0:i] G[0:i, i].
__global__ __launch_bounds__(256) void dc_tfactor_kernel(const DcTable tab)
{
    __shared__ float G[64][65], T[64][65], taus[64];
    int local;
    const DcProb &pr = dc_locate(tab, local);
    if (pr.n <= kDcLeaf) return;
    const DcWs ws(pr.ws, pr.n);
    const int n = pr.n, ld = dc_ld(n), j0 = 64 * local;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lk = lane >> 4;
    floatx4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto row = [&](int j, int i) {          // four elements of reflector j (rows from n - 2 on hold none)
        floatx4 x = {0.f, 0.f, 0.f, 0.f};
        if (j < n - 2 && i < ld) x = *reinterpret_cast<const floatx4 *>(ws.A + (long)j * ld + i);
        return x;
    };
    for (int i = j0 + 4 * lk; i < n + 4 * lk; i += 16) {
        const floatx4 a = row(j0 + 16 * w + lr, i);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const floatx4 b = row(j0 + 16 * t + lr, i);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) G[16 * w + 4 * lk + v][16 * t + lr] = acc[t][v];
    for (int e = tid; e < 64 * 64; e += 256) T[e >> 6][e & 63] = 0.f;
    __syncthreads();
    if (tid < 64) taus[tid] = ws.tau[j0 + tid];
    __syncthreads();
    const int ra = tid >> 2, part = tid & 3;          // four threads sum a row
    for (int i = 0; i < 64; ++i) {
        const float tau = taus[i];
        float s = 0.f;
#pragma unroll 4
        for (int b = (ra & ~3) + part; b < i; b += 4) s = __builtin_fmaf(T[ra][b], G[b][i], s);    // (T is zero below its diagonal)
        s += dc_dpp<0xB1, 0xf>(s);                    // quad_perm 1 0 3 2, then 2 3 0 1
        s += dc_dpp<0x4E, 0xf>(s);
        if (part == 0 && ra <= i) T[ra][i] = ra < i ? -tau * s : tau;
        __syncthreads();
    }
    float *out = ws.T + (size_t)local * 64 * 64;
    for (int e = tid; e < 64 * 64; e += 256) out[e] = T[e >> 6][e & 63];
}

// Q^T = V (I - Y T^T Y^T) ..., 16 MT eigenvectors per workgroup in LDS, the last block of reflectors first; then Q and v.
template <int MT>
__device__ __forceinline__ void dc_back(const DcProb &pr, int local, float *lds)
{
    constexpr int R = 16 * MT, PP = 68;
    const DcWs ws(pr.ws, pr.n);
    const int n = pr.n, ld = dc_ld(n), r0 = R * local;
    const int px = (ld + 15) / 16 * 16 + 4;              // pitch of a vector: whole chunks of 16, 4 mod 16
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lk = lane >> 4;
    float *X = lds, *P = X + R * px, *P2 = P + R * PP;
    const float *V = ws.V(dc_levels(n));
    for (int e = tid; e < R * (px / 4); e += 256) {
        const int r = e / (px / 4), c = 4 * (e - r * (px / 4));
        floatx4 x = {0.f, 0.f, 0.f, 0.f};
        if (r0 + r < n && c < ld) x = *reinterpret_cast<const floatx4 *>(V + (long)(r0 + r) * ld + c);
#pragma unroll
        for (int q = 0; q < 4; ++q) X[r * px + c + q] = c + q < n ? x[q] : 0.f;
    }
    __syncthreads();
    for (int b = (n - 3) / 64; b >= 0; --b) {
        const int j0 = 64 * b;
        // P = X Y: wavefront w takes 16 reflectors
        floatx4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int j = j0 + 16 * w + lr;
        const bool have = j < n - 2;
        const float *yr = ws.A + (long)(have ? j : 0) * ld;
#pragma unroll 4
        for (int i0 = j0; i0 < ld; i0 += 16) {
            const int i = i0 + 4 * lk;
            floatx4 y = *reinterpret_cast<const floatx4 *>(yr + (i < ld ? i : 0));
            if (!have || i >= ld) y = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const floatx4 x = *reinterpret_cast<const floatx4 *>(X + (16 * m + lr) * px + i);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc[m], 0, 0, 0);
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) P[(16 * m + 4 * lk + v) * PP + 16 * w + lr] = acc[m][v];
        __syncthreads();
        // P2 = P T^T
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        const float *tr = ws.T + (size_t)b * 64 * 64 + (16 * w + lr) * 64;
#pragma unroll
        for (int a0 = 0; a0 < 64; a0 += 16) {
            const floatx4 t = *reinterpret_cast<const floatx4 *>(tr + a0 + 4 * lk);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const floatx4 p = *reinterpret_cast<const floatx4 *>(P + (16 * m + lr) * PP + a0 + 4 * lk);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[e], t[e], acc[m], 0, 0, 0);
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) P2[(16 * m + 4 * lk + v) * PP + 16 * w + lr] = acc[m][v];
        __syncthreads();
        // X -= P2 Y^T: 64 columns of X at a time, lanes four neighbours each
        for (int i0 = j0 + 64 * w; i0 < ld; i0 += 256) {
            const int i = i0 + 4 * lr;
            floatx4 d[MT][4];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < 4; ++t) d[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int a0 = 0; a0 < 64; a0 += 4) {
                const int a = j0 + a0 + lk;
                floatx4 y = *reinterpret_cast<const floatx4 *>(ws.A + (long)(a < n - 2 ? a : 0) * ld + (i < ld ? i : 0));
                if (a >= n - 2 || i >= ld) y = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const float p = P2[(16 * m + lr) * PP + a0 + lk];
#pragma unroll
                    for (int t = 0; t < 4; ++t) d[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(p, y[t], d[m][t], 0, 0, 0);
                }
            }
            if (i < ld) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        floatx4 *x = reinterpret_cast<floatx4 *>(X + (16 * m + 4 * lk + v) * px + i);
                        *x -= floatx4{d[m][0][v], d[m][1][v], d[m][2][v], d[m][3][v]};
                    }
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < R * n; e += 256) {
        const int i = e / R, r = e - i * R;
        if (r0 + r < n) pr.Q[(long)i * n + r0 + r] = X[r * px + i];
    }
    if (tid < R && r0 + tid < n) pr.v[r0 + tid] = (float)ws.d[r0 + tid];
}

// 32 vectors per workgroup up to order 320 (59 KB of LDS), 16 above (50 KB up to 640, 91 KB up to 1280)
template <int MT, int NMAX>
__global__ __launch_bounds__(256) void dc_back_kernel(const DcTable tab)
{
    __shared__ __attribute__((aligned(16))) float lds[16 * MT * (NMAX + 4 + 2 * 68)];
    int local;
    const DcProb &pr = dc_locate(tab, local);
    dc_back<MT>(pr, local, lds);
}

}  // namespace kfac
