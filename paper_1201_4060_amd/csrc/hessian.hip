// Second derivatives of the interpolant, with u and grad u.
//
// Section 2: the l-th derivative of the interpolant on a cell uses the matrix
// M^(l) = M D^l; here l = 2 gives the weights w''_j(t).  In three dimensions
// (Section 3) the mixed derivative d2/dx_i dx_j takes the first-derivative
// weights on axes i and j, and d2/dx_i^2 the second-derivative weights on
// axis i; every factor carries the chain factor n/L of its axis.  The
// particles are binned as for the evaluation (tiles of 8^3 cells) and
// gathered from an LDS copy of each tile's block of the grid (or, for classes
// without a tiled body, one lane per particle straight from the grid), the
// contraction reducing axis 2 first, then axis 1, then axis 0 (the Table 1
// idea), with six per-plane partial sums per component instead of three.
//
// Output per particle p and component c: u[p][c], grad[p][c][d] and
// hess[p][c][m] = d2 u_c / dx_i dx_j for (i, j) = (0,0), (0,1), (0,2), (1,1),
// (1,2), (2,2) in that order.
#include <algorithm>

#include "gather.hpp"

namespace bsi {

namespace {

constexpr int HESS_B = 256;

// M^(2)[r][c] = (c+1)(c+2) M[r][c+2] (M D^2, Section 2), at compile time.
template <int N>
struct BSpline2 {
    double M2[N][N];
    constexpr BSpline2() : M2{} {
        for (int r = 0; r < N; ++r)
            for (int c = 0; c < N; ++c)
                M2[r][c] = (c + 2 < N) ? double((c + 1) * (c + 2) * bspline_numer(N, r, c + 2)) /
                                             double(fact_ll(N - 1))
                                       : 0.0;
    }
};

// w''_j(t) = sum_i M^(2)[j][i] t^i (Horner)
template <int N, typename AT>
__device__ __forceinline__ void bspline_weights2(AT t, AT* wdd) {
    constexpr BSpline2<N> B{};
#pragma unroll
    for (int j = 0; j < N; ++j) {
        AT acc = AT(B.M2[j][N - 3]);
#pragma unroll
        for (int i = N - 4; i >= 0; --i) acc = fused(acc, t, AT(B.M2[j][i]));
        wdd[j] = acc;
    }
}

struct HessArgs {
    const void* grid;
    const void* binned;        // the particles in binned order (RawParticle)
    const uint32_t* perm;      // particle of every binned slot
    long P;
    int n0, n1, n2, P1;
    int pitch2;
    double ih0, ih1, ih2;
    void* u;
    void* grad;  // or nullptr
    void* hess;
    unsigned long long* nonfinite;
    ItemSource src;            // work items (tiled kernel)
};

// Cell and weights (value, first and second derivative, chain factors
// included) of a binned particle; false when it has no cell.
template <int N, typename AT>
__device__ __forceinline__ bool hess_setup(const HessArgs& a, const RawParticle<AT>& raw, int* cell, AT (*w)[N],
                                           AT (*wd)[N], AT (*wdd)[N]) {
    const int n[3] = {a.n0, a.n1, a.n2};
    const double ih[3] = {a.ih0, a.ih1, a.ih2};
    AT t[3];
    if (!locate(raw, n, ih, cell, t)) return false;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        bspline_weights<N, AT>(t[d], w[d], wd[d]);
        bspline_weights2<N, AT>(t[d], wdd[d]);
        const AT s = AT(ih[d]);
        const AT s2 = AT(ih[d] * ih[d]);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            wd[d][k] *= s;
            wdd[d][k] *= s2;
        }
    }
    return true;
}

// One lane per binned slot j; results are written at the particle's index.
template <int N, typename CT, int C>
__global__ __launch_bounds__(HESS_B) void k_gather_hess(HessArgs a) {
    using AT = typename Acc<CT>::type;
    const long j = long(blockIdx.x) * HESS_B + threadIdx.x;
    if (j >= a.P) return;
    const long p = long(a.perm[j]);
    RawParticle<AT> raw;
    raw.load(a.binned, j);
    int cell[3];
    AT w[3][N], wd[3][N], wdd[3][N];
    const bool ok = hess_setup<N, AT>(a, raw, cell, w, wd, wdd);
    AT* u = static_cast<AT*>(a.u) + p * C;
    AT* g = a.grad ? static_cast<AT*>(a.grad) + p * C * 3 : nullptr;
    AT* h = static_cast<AT*>(a.hess) + p * C * 6;
    if (!ok) {
        const AT nan = AT(__builtin_nan(""));
        for (int c = 0; c < C; ++c) u[c] = nan;
        if (g)
            for (int c = 0; c < 3 * C; ++c) g[c] = nan;
        for (int c = 0; c < 6 * C; ++c) h[c] = nan;
        atomicAdd(a.nonfinite, 1ull);
        return;
    }
    const CT* base = static_cast<const CT*>(a.grid) + (long(cell[0]) * a.P1 + cell[1]) * a.pitch2 +
                     long(cell[2]) * C;
    const long rowA = long(a.P1) * a.pitch2;
    const long rowB = a.pitch2;
    AT U[C], G0[C], G1[C], G2[C], H00[C], H01[C], H02[C], H11[C], H12[C], H22[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        U[c] = G0[c] = G1[c] = G2[c] = H00[c] = H01[c] = H02[c] = H11[c] = H12[c] = H22[c] = AT(0);
#pragma unroll 1
    for (int ia = 0; ia < N; ++ia) {
        AT v[C], v1[C], v2[C], v11[C], v12[C], v22[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = v1[c] = v2[c] = v11[c] = v12[c] = v22[c] = AT(0);
#pragma unroll
        for (int ib = 0; ib < N; ++ib) {
            const CT* r = base + ia * rowA + ib * rowB;
            AT tr[C], trd[C], trdd[C];
#pragma unroll
            for (int c = 0; c < C; ++c) tr[c] = trd[c] = trdd[c] = AT(0);
#pragma unroll
            for (int e = 0; e < N; ++e) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const AT val = widen<CT, AT>(r[e * C + c]);
                    tr[c] += w[2][e] * val;
                    trd[c] += wd[2][e] * val;
                    trdd[c] += wdd[2][e] * val;
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                v[c] += w[1][ib] * tr[c];
                v1[c] += wd[1][ib] * tr[c];
                v2[c] += w[1][ib] * trd[c];
                v11[c] += wdd[1][ib] * tr[c];
                v12[c] += wd[1][ib] * trd[c];
                v22[c] += w[1][ib] * trdd[c];
            }
        }
        // the axis-0 weights of plane ia, picked without dynamic indexing
        AT w0 = w[0][0], wd0 = wd[0][0], wdd0 = wdd[0][0];
#pragma unroll
        for (int k = 1; k < N; ++k) {
            w0 = ia == k ? w[0][k] : w0;
            wd0 = ia == k ? wd[0][k] : wd0;
            wdd0 = ia == k ? wdd[0][k] : wdd0;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            U[c] += w0 * v[c];
            G0[c] += wd0 * v[c];
            G1[c] += w0 * v1[c];
            G2[c] += w0 * v2[c];
            H00[c] += wdd0 * v[c];
            H01[c] += wd0 * v1[c];
            H02[c] += wd0 * v2[c];
            H11[c] += w0 * v11[c];
            H12[c] += w0 * v12[c];
            H22[c] += w0 * v22[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        u[c] = U[c];
        if (g) {
            g[3 * c + 0] = G0[c];
            g[3 * c + 1] = G1[c];
            g[3 * c + 2] = G2[c];
        }
        h[6 * c + 0] = H00[c];
        h[6 * c + 1] = H01[c];
        h[6 * c + 2] = H02[c];
        h[6 * c + 3] = H11[c];
        h[6 * c + 4] = H12[c];
        h[6 * c + 5] = H22[c];
    }
}

// Sums over axis-0 planes: u, the three first and six second derivatives.
template <typename AT, int C>
struct HessSums {
    AT s[10][C];
};

// Planes k = 0..NP-1 with axis-0 weights w0[k], wd0[k], wdd0[k] and rows
// row(k, ib), accumulated in plane order into out (axis 2 first, then 1).
template <int N, typename CT, typename AT, int C, int NP, typename RowFn>
__device__ __forceinline__ void hess_planes(const AT* w0, const AT* wd0, const AT* wdd0, const AT (*w)[N],
                                            const AT (*wd)[N], const AT (*wdd)[N], RowFn row,
                                            HessSums<AT, C>& out) {
#pragma unroll
    for (int m = 0; m < 10; ++m)
#pragma unroll
        for (int c = 0; c < C; ++c) out.s[m][c] = AT(0);
#pragma unroll 1
    for (int k = 0; k < NP; ++k) {
        AT a0 = w0[0], d0 = wd0[0], dd0 = wdd0[0];
#pragma unroll
        for (int q = 1; q < NP; ++q) {
            a0 = k == q ? w0[q] : a0;
            d0 = k == q ? wd0[q] : d0;
            dd0 = k == q ? wdd0[q] : dd0;
        }
        AT v[C], v1[C], v2[C], v11[C], v12[C], v22[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = v1[c] = v2[c] = v11[c] = v12[c] = v22[c] = AT(0);
#pragma unroll
        for (int ib = 0; ib < N; ++ib) {
            const CT* r = row(k, ib);
            CT raw[N * C];
            if constexpr (sizeof(CT) == 2 && (N * C) % 2 == 0) {
                // BF16 rows start on 2-byte boundaries: aligned dword reads and
                // a funnel shift by the misalignment, as in the gather
                typedef const __attribute__((address_space(3))) uint16_t lds_u16;
                typedef const __attribute__((address_space(3))) uint32_t lds_u32;
                lds_u16* lr = (lds_u16*)(r);
                const uint32_t mis = uint32_t(reinterpret_cast<uintptr_t>(lr)) & 2u;
                lds_u32* d = (lds_u32*)(lr - (mis >> 1));
                constexpr int ND = N * C / 2 + 1;
                uint32_t dw[ND];
#pragma unroll
                for (int q = 0; q < ND; ++q) dw[q] = d[q];
#pragma unroll
                for (int q = 0; q < N * C / 2; ++q) {
                    const uint32_t v = __builtin_amdgcn_alignbit(dw[q + 1], dw[q], mis * 8u);
                    raw[2 * q] = CT(v & 0xffffu);
                    raw[2 * q + 1] = CT(v >> 16);
                }
            } else {
#pragma unroll
                for (int e = 0; e < N * C; ++e) raw[e] = r[e];
            }
            AT tr[C], trd[C], trdd[C];
#pragma unroll
            for (int c = 0; c < C; ++c) tr[c] = trd[c] = trdd[c] = AT(0);
#pragma unroll
            for (int e = 0; e < N; ++e) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const AT val = widen<CT, AT>(raw[e * C + c]);
                    tr[c] += w[2][e] * val;
                    trd[c] += wd[2][e] * val;
                    trdd[c] += wdd[2][e] * val;
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                v[c] += w[1][ib] * tr[c];
                v1[c] += wd[1][ib] * tr[c];
                v2[c] += w[1][ib] * trd[c];
                v11[c] += wdd[1][ib] * tr[c];
                v12[c] += wd[1][ib] * trd[c];
                v22[c] += w[1][ib] * trdd[c];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            out.s[0][c] += a0 * v[c];
            out.s[1][c] += d0 * v[c];
            out.s[2][c] += a0 * v1[c];
            out.s[3][c] += a0 * v2[c];
            out.s[4][c] += dd0 * v[c];
            out.s[5][c] += d0 * v1[c];
            out.s[6][c] += d0 * v2[c];
            out.s[7][c] += a0 * v11[c];
            out.s[8][c] += a0 * v12[c];
            out.s[9][c] += a0 * v22[c];
        }
    }
}

// u, grad u (if requested) and hess of particle p from the two halves of the
// axis-0 sum.
template <typename AT, int C>
__device__ __forceinline__ void hess_store(const HessArgs& a, long p, const HessSums<AT, C>& lo,
                                           const HessSums<AT, C>& hi) {
    AT* u = static_cast<AT*>(a.u) + p * C;
    AT* h = static_cast<AT*>(a.hess) + p * C * 6;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        u[c] = lo.s[0][c] + hi.s[0][c];
#pragma unroll
        for (int m = 0; m < 6; ++m) h[6 * c + m] = lo.s[4 + m][c] + hi.s[4 + m][c];
    }
    if (a.grad) {
        AT* g = static_cast<AT*>(a.grad) + p * C * 3;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int d = 0; d < 3; ++d) g[3 * c + d] = lo.s[1 + d][c] + hi.s[1 + d][c];
    }
}

template <typename AT, int C>
__device__ __forceinline__ void hess_nan(const HessArgs& a, long p) {
    const AT nan = AT(__builtin_nan(""));
    AT* u = static_cast<AT*>(a.u) + p * C;
    AT* h = static_cast<AT*>(a.hess) + p * C * 6;
    for (int c = 0; c < C; ++c) u[c] = nan;
    for (int c = 0; c < 6 * C; ++c) h[c] = nan;
    if (a.grad) {
        AT* g = static_cast<AT*>(a.grad) + p * C * 3;
        for (int c = 0; c < 3 * C; ++c) g[c] = nan;
    }
}

// What the tiled kernel does with one particle: u, grad u and the second
// derivatives, on two lanes (one half of the axis-0 sum each, combined by a lane
// exchange) or one.
template <int N_, typename CT_, int C_>
struct HessGather {
    static constexpr int N = N_, C = C_, T = 8;
    using CT = CT_;
    using AT = typename Acc<CT>::type;
    using G = TileGeom<N, CT, C, T, false>;   // rows packed densely (hess_planes reads them)
    using Args = HessArgs;
    struct Weights {
        AT w[3][N], wd[3][N], wdd[3][N];
    };
    template <int W>
    __device__ __forceinline__ static int lanes(uint32_t count) {
        return count <= uint32_t(W * 32) ? 2 : 1;
    }
    struct Shared {};
    __device__ __forceinline__ static void init(const Args&, Shared*) {}
    __device__ __forceinline__ static void setup(const Args& a, const RawParticle<AT>& raw, int, const LaneRole&,
                                                 int* cell, Weights& k, Shared*) {
        hess_setup<N, AT>(a, raw, cell, k.w, k.wd, k.wdd);   // finite by construction of the tile
    }
    template <typename RowFn>
    __device__ __forceinline__ static void eval(const Args& a, long p, bool active, int lanes, int part,
                                                const Weights& k, RowFn rows) {
        if (lanes == 2) {
            const int ia0 = part * (N / 2);
            AT w0s[N / 2], wd0s[N / 2], wdd0s[N / 2];
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                w0s[i] = part ? k.w[0][N / 2 + i] : k.w[0][i];
                wd0s[i] = part ? k.wd[0][N / 2 + i] : k.wd[0][i];
                wdd0s[i] = part ? k.wdd[0][N / 2 + i] : k.wdd[0][i];
            }
            HessSums<AT, C> mine, other;
            hess_planes<N, CT, AT, C, N / 2>(w0s, wd0s, wdd0s, k.w, k.wd, k.wdd,
                                             [&](int i, int ib) { return rows(ia0 + i, ib); }, mine);
#pragma unroll
            for (int m = 0; m < 10; ++m)
#pragma unroll
                for (int c = 0; c < C; ++c) other.s[m][c] = quad_lane<QUAD_XOR1>(mine.s[m][c]);
            if (active && part == 0) hess_store<AT, C>(a, p, mine, other);
        } else {
            HessSums<AT, C> lo, hi;
            hess_planes<N, CT, AT, C, N / 2>(k.w[0], k.wd[0], k.wdd[0], k.w, k.wd, k.wdd, rows, lo);
            hess_planes<N, CT, AT, C, N / 2>(k.w[0] + N / 2, k.wd[0] + N / 2, k.wdd[0] + N / 2, k.w, k.wd, k.wdd,
                                             [&](int i, int ib) { return rows(N / 2 + i, ib); }, hi);
            if (active) hess_store<AT, C>(a, p, lo, hi);
        }
    }
    template <int B>
    __device__ __forceinline__ static void nonfinite(const Args& a, uint32_t count, uint32_t start) {
        for (uint32_t j = threadIdx.x; j < count; j += B) hess_nan<AT, C>(a, long(a.perm[start + j]));
        if (threadIdx.x == 0) atomicAdd(a.nonfinite, (unsigned long long)count);
    }
};

constexpr int HESS_TB = 64;           // threads per workgroup of the tiled kernel
constexpr uint32_t HESS_ROUNDS = 4;   // rounds of one wavefront per work item

// LDS-tiled variant: the evaluation's tiled gather with these sums.
template <int N, typename CT, int C>
__global__ __launch_bounds__(HESS_TB) void k_gather_hess_tiled(HessArgs a) {
    using K = HessGather<N, CT, C>;
    __shared__ u32x4 lds[tile_lds_bytes<K>() / 16];
    tiled_gather<K, HESS_TB>([&](uint32_t, HessArgs& x) { x = a; }, a.src, true, lds,
                             nullptr, nullptr);
}

template <typename CT>
bool hess_tiled_ok(int N, int C) {
    // FP64 three-component order 6 spills registers in the tiled body: direct
    if (sizeof(CT) == 8 && N == 6 && C == 3) return false;
    auto ok = [](auto g) { return decltype(g)::BYTES <= 65536 && decltype(g)::ALIGNED; };
    if (N == 4) return C == 1 ? ok(TileGeom<4, CT, 1, 8, false>{}) : ok(TileGeom<4, CT, 3, 8, false>{});
    return C == 1 ? ok(TileGeom<6, CT, 1, 8, false>{}) : ok(TileGeom<6, CT, 3, 8, false>{});
}

// Persistent launch: as many workgroups as stay resident (the kernel's
// occupancy, asked once per instance) on every CU.
template <int N, typename CT, int C>
void launch_hess_tiled(int num_cus, hipStream_t s, const HessArgs& a) {
    auto k = k_gather_hess_tiled<N, CT, C>;
    static unsigned per_cu = 0;
    static std::once_flag once;
    std::call_once(once, [&] {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k, HESS_TB, 0) != hipSuccess || v < 1) v = 1;
        per_cu = unsigned(v);
    });
    hipLaunchKernelGGL(k, dim3(per_cu * unsigned(std::max(num_cus, 1))), dim3(HESS_TB), 0, s, a);
}

template <typename CT>
void launch_hess_tiled_ct(int N, int C, int num_cus, hipStream_t s, const HessArgs& a) {
    if (N == 4) {
        if (C == 1) launch_hess_tiled<4, CT, 1>(num_cus, s, a);
        else launch_hess_tiled<4, CT, 3>(num_cus, s, a);
    } else {
        if (C == 1) launch_hess_tiled<6, CT, 1>(num_cus, s, a);
        else launch_hess_tiled<6, CT, 3>(num_cus, s, a);
    }
}

template <typename CT>
void launch_hess_ct(int N, int C, unsigned nb, hipStream_t s, const HessArgs& a) {
    if (N == 4) {
        if (C == 1) hipLaunchKernelGGL((k_gather_hess<4, CT, 1>), dim3(nb), dim3(HESS_B), 0, s, a);
        else hipLaunchKernelGGL((k_gather_hess<4, CT, 3>), dim3(nb), dim3(HESS_B), 0, s, a);
    } else {
        if (C == 1) hipLaunchKernelGGL((k_gather_hess<6, CT, 1>), dim3(nb), dim3(HESS_B), 0, s, a);
        else hipLaunchKernelGGL((k_gather_hess<6, CT, 3>), dim3(nb), dim3(HESS_B), 0, s, a);
    }
}

}  // namespace

bsi_status hessian_run(bsi_field* f, const double* pos, int64_t P, void* u, void* grad, void* hess,
                       hipStream_t s) {
    BSI_CHECK(f->basis == BSI_BASIS_BSPLINE && (f->N == 4 || f->N == 6), BSI_E_UNSUPPORTED,
              "second derivatives are implemented for B-spline fields of orders 4 and 6");
    if (P == 0) return BSI_OK;
    // binned by tiles of 8 cells (at least n/256, so that the bucket
    // table has at most 2^24 entries), for locality of the stencil reads
    const int nmax = std::max(f->n[0], std::max(f->n[1], f->n[2]));
    const int tile = std::max(8, (nmax + 255) / 256);
    const int coef = f->desc.coef;
    const bool tiled = tile == 8 && (coef == BSI_F64   ? hess_tiled_ok<double>(f->N, f->C)
                                     : coef == BSI_F32 ? hess_tiled_ok<float>(f->N, f->C)
                                                       : hess_tiled_ok<uint16_t>(f->N, f->C));
    const BinLayout l = bin_layout(f, long(P), tile, tiled ? uint32_t(HESS_TB) * HESS_ROUNDS : 0u);
    void* ws = nullptr;
    BSI_TRY(get_workspace(f->ctx->eval_ws, s, l.bytes, &ws));
    BSI_TRY(bin_run(f, pos, long(P), tile, l, ws, s));
    const BinArrays b = bin_arrays(f, long(P), tile, l, ws);
    HessArgs a;
    a.grid = f->grid;
    a.binned = b.binned;
    a.perm = b.perm;
    a.P = long(P);
    a.n0 = f->n[0];
    a.n1 = f->n[1];
    a.n2 = f->n[2];
    a.P1 = f->P[1];
    a.pitch2 = f->pitch2;
    a.ih0 = f->inv_h[0];
    a.ih1 = f->inv_h[1];
    a.ih2 = f->inv_h[2];
    a.u = u;
    a.grad = grad;
    a.hess = hess;
    a.nonfinite = f->counters;
    a.src = item_source(b);
    {
        StageTimer tm(f->ctx, "gather_hess", s);
        if (tiled) {
            const int cus = f->ctx->num_cus;
            if (coef == BSI_F64) launch_hess_tiled_ct<double>(f->N, f->C, cus, s, a);
            else if (coef == BSI_F32) launch_hess_tiled_ct<float>(f->N, f->C, cus, s, a);
            else launch_hess_tiled_ct<uint16_t>(f->N, f->C, cus, s, a);
        } else {
            const unsigned nb = unsigned((P + HESS_B - 1) / HESS_B);
            if (coef == BSI_F64) launch_hess_ct<double>(f->N, f->C, nb, s, a);
            else if (coef == BSI_F32) launch_hess_ct<float>(f->N, f->C, nb, s, a);
            else launch_hess_ct<uint16_t>(f->N, f->C, nb, s, a);
        }
    }
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

}  // namespace bsi
