// Prefilter on the GPU: symbol multiply + one inverse 3D real FFT (Section 7).
//
// Pass A  (axis 0)  reads the caller's half spectrum uhat[c][k0][k1][k2],
//                   multiplies it by c(k0) c(k1) c(k2) in FP64, casts to the
//                   working precision T and does the inverse complex FFT along
//                   k0, writing the work buffer (same layout).
// Pass B  (axis 1)  inverse complex FFT along k1, in place.
// Pass C  (axis 2)  complex-to-real inverse FFT of each k2 line (length n2/2
//                   complex FFT after the standard even/odd twist), cast to the
//                   storage type and written to the ghost-padded, component-
//                   interleaved coefficient grid.
//
// Every line transform is a Stockham autosort FFT: each stage has every thread
// load its radix-R butterflies into registers, apply twiddles from a table of
// exp(+2 pi i m / len) (computed on the host in FP64), do the radix-R DFT and
// store to the self-sorted positions.  Pass C holds its lines in LDS throughout.  In
// passes A and B a workgroup transforms W adjacent lines of a strided axis, so that
// each global row access covers W consecutive elements; the lines stay in registers
// and only change hands through LDS between two stages.
#include "common.hpp"
#include "device.hpp"

// No product is fused into a sum but where fused() says so: left to the compiler,
// instances of different lengths and types fuse differently, and a transform's last
// bits (and with them the BF16 rounding of its FP32 result) would depend on which
// instance ran.
#pragma clang fp contract(off)

namespace bsi {

template <typename T>
__device__ __forceinline__ cplx<T> cadd(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> csub(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }
// a times the twiddle b.  Of the two products of the imaginary part the first is
// rounded before the sum and the second is not; turned: the other way round (turned()
// below; in pass C for axes of 32 points).
template <typename T>
__device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b, bool turned = false) {
    return {fused(a.x, b.x, -(a.y * b.y)), turned ? fused(a.x, b.y, a.y * b.x) : fused(a.y, b.x, a.x * b.y)};
}
template <typename T>
__device__ __forceinline__ cplx<T> cmul_i(cplx<T> a) { return {-a.y, a.x}; }  // i * a

// Inverse (sign +) DFT of length R in registers.
template <typename T>
__device__ __forceinline__ void dft2(cplx<T>* v) {
    cplx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}
template <typename T>
__device__ __forceinline__ void dft3(cplx<T>* v) {
    const T h = T(0.86602540378443864676372317075294);  // sin(2 pi / 3)
    cplx<T> s = cadd(v[1], v[2]);
    cplx<T> d = csub(v[1], v[2]);
    cplx<T> m = {fused(T(-0.5), s.x, v[0].x), fused(T(-0.5), s.y, v[0].y)};
    v[0] = cadd(v[0], s);
    v[1] = {fused(-h, d.y, m.x), fused(h, d.x, m.y)};  // m + i h d
    v[2] = {fused(h, d.y, m.x), fused(-h, d.x, m.y)};
}
template <typename T>
__device__ __forceinline__ void dft4(cplx<T>* v) {
    cplx<T> s0 = cadd(v[0], v[2]), s1 = csub(v[0], v[2]);
    cplx<T> s2 = cadd(v[1], v[3]), s3 = cmul_i(csub(v[1], v[3]));
    v[0] = cadd(s0, s2);
    v[2] = csub(s0, s2);
    v[1] = cadd(s1, s3);
    v[3] = csub(s1, s3);
}
template <typename T>
__device__ __forceinline__ void dft8(cplx<T>* v) {
    const T r2 = T(0.70710678118654752440084436210485);
    cplx<T> e[4] = {v[0], v[2], v[4], v[6]};
    cplx<T> o[4] = {v[1], v[3], v[5], v[7]};
    dft4(e);
    dft4(o);
    o[1] = {o[1].x - o[1].y, o[1].x + o[1].y};   // r2 o1 = o1 e^{+i pi/4}
    o[2] = cmul_i(o[2]);                         // o2 e^{+i pi/2}
    o[3] = {-(o[3].x + o[3].y), o[3].x - o[3].y};  // r2 o3 = o3 e^{+3i pi/4}
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q & 1) {
            v[q] = {fused(r2, o[q].x, e[q].x), fused(r2, o[q].y, e[q].y)};
            v[q + 4] = {fused(-r2, o[q].x, e[q].x), fused(-r2, o[q].y, e[q].y)};
        } else {
            v[q] = cadd(e[q], o[q]);
            v[q + 4] = csub(e[q], o[q]);
        }
    }
}
template <typename T, int R>
__device__ __forceinline__ void dft(cplx<T>* v) {
    if constexpr (R == 2) dft2(v);
    else if constexpr (R == 3) dft3(v);
    else if constexpr (R == 4) dft4(v);
    else dft8(v);
}

template <int REM>
struct Radix {
    static constexpr int value = (REM % 3 == 0) ? 3 : (REM % 8 == 0) ? 8 : (REM % 4 == 0) ? 4 : 2;
};

// Place of element i of an LDS line of FP64 values, one spare place every 16: the
// lanes of a line write a stage's results at strides of 2 to 64 elements, which
// would otherwise meet in a few banks (pass C at 128 x 192 lines of 256 FP64: 81 ->
// 73 us; with FP32 values the index arithmetic costs more, 512^3: 745 -> 775).
template <typename T>
__host__ __device__ constexpr int spread(int i) {
    return sizeof(T) == 8 ? i + (i >> 4) : i;
}
template <typename T>
constexpr int spread_len(int n) {
    return spread<T>(n - 1) + 1;
}

// Stockham stages NS.. of an inverse FFT of length LEN on one LDS line
// (spread).
// tw[m * TWS] = exp(+2 pi i m / LEN).  All threads of the block must call this
// with the same template arguments (it contains block barriers).
template <typename T, int LEN, int TEAM, int NS, int TWS>
__device__ __forceinline__ void fft_stages(cplx<T>* buf, const cplx<T>* tw, int lane) {
    if constexpr (NS < LEN) {
        constexpr int R = Radix<LEN / NS>::value;
        constexpr int NB = LEN / R;
        constexpr int PER = (NB + TEAM - 1) / TEAM;
        constexpr int TSTEP = LEN / (NS * R);
        cplx<T> v[PER][R];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int j = lane + q * TEAM;
            if (PER * TEAM == NB || j < NB) {
                const int k = j % NS;
#pragma unroll
                for (int r = 0; r < R; ++r) v[q][r] = buf[spread<T>(j + r * NB)];
                if constexpr (NS > 1) {
#pragma unroll
                    for (int r = 1; r < R; ++r) v[q][r] = cmul(v[q][r], tw[r * k * TSTEP * TWS], LEN == 16);
                }
                dft<T, R>(v[q]);
            }
        }
        lds_barrier();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int j = lane + q * TEAM;
            if (PER * TEAM == NB || j < NB) {
                const int k = j % NS;
                const int base = (j / NS) * NS * R + k;
#pragma unroll
                for (int r = 0; r < R; ++r) buf[spread<T>(base + r * NS)] = v[q][r];
            }
        }
        lds_barrier();
        fft_stages<T, LEN, TEAM, NS * R, TWS>(buf, tw, lane);
    }
}

// The most threads a line can have when a thread that holds the rows a0 + q TEAM is
// to hold whole butterflies of every stage: the largest power of two that divides
// LEN / R for every radix R in turn.
constexpr int common_pow2(int a, int b) {
    int t = 1;
    while (a % (2 * t) == 0 && b % (2 * t) == 0) t *= 2;
    return t;
}
template <int LEN, int NS = 1>
constexpr int line_team() {
    if constexpr (NS == LEN) return LEN;
    else return common_pow2(LEN / Radix<LEN / NS>::value, line_team<LEN, NS * Radix<LEN / NS>::value>());
}

// A strided-pass workgroup: W lines of TEAM threads.  Longer contiguous row segments
// (W elements) are better for HBM and two workgroups a CU let one load while the
// other transforms, so a workgroup gets half of the CU's LDS, or nearly all of it
// where fewer than 8 lines would fit (FP64, 1024 points).
template <typename T, int LEN>
struct StridedCfg {
    static constexpr int LP = LEN + 1;                     // odd: the lines start in different banks
    static constexpr int LINE = LP * int(sizeof(cplx<T>));
    static constexpr int TW = LEN * int(sizeof(cplx<T>));
    static constexpr int KB = (80 * 1024 - TW) / LINE < 8 ? 150 : 80;
    static constexpr int fit = (KB * 1024 - TW) / LINE;
    static constexpr int W = fit >= 32 ? 32 : fit >= 16 ? 16 : 8;
    static constexpr int MOST = 512 / W;
    static constexpr int TEAM = MOST < line_team<LEN>() ? MOST : line_team<LEN>();
    static constexpr int THREADS = W * TEAM;
    static constexpr int PER = LEN / TEAM;                 // values per thread
    // wavefronts per SIMD to compile for
    static constexpr int WAVES = THREADS < 512 ? 1 : KB == 80 ? 4 : 2;
};

// The butterflies [lo, hi) of the stage after transforms of length ns whose twiddle
// products are turned (cmul).  Either way is as exact.  But a last bit that differs
// here rounds one value in 10^4 of a BF16 grid to its other neighbour, which the
// interpolated values show (5e-5 of their norm at 1024^3), so the ways are part of
// the result and are kept as stored grids have them: turned where a thread's
// butterfly, of those `team` apart, meets an earlier one's twiddles again, `team`
// being another number of threads than the present one in three passes; none in the
// last column of the half spectrum where n2/2 is a multiple of 32 (k_fft_axis:
// ALONE; that column is then a block of its own).
struct Turned {
    int lo, hi;
};
template <typename T, int LEN, int TEAM, bool FIRST>
constexpr Turned turned(int ns) {
    constexpr bool dbl = sizeof(T) == 8;
    if (LEN % 3 == 0) return {0, 0};
    if (FIRST && !dbl && LEN == 1024) return ns == 8 ? Turned{32, 128} : ns == 64 ? Turned{64, 96} : Turned{0, 0};
    const int team = FIRST && !dbl && LEN == 512 ? 16 : !FIRST && dbl && LEN == 1024 ? 256 : TEAM;
    return {ns > team ? ns : team, LEN};
}

// The thread's butterflies of the stage that follows transforms of length NS, in
// place: butterfly m is v[m + r BPT], r < R.
template <typename T, int LEN, int TEAM, bool FIRST, int R, int NS>
__device__ __forceinline__ void butterflies(cplx<T>* v, const cplx<T>* tw, int a0, bool last) {
    constexpr int BPT = LEN / R / TEAM;
    constexpr Turned U = turned<T, LEN, TEAM, FIRST>(NS);
    static_assert(BPT * R * TEAM == LEN, "whole butterflies per thread");
#pragma unroll
    for (int m = 0; m < BPT; ++m) {
        cplx<T> x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = v[m + r * BPT];
        if constexpr (NS > 1) {
            const int k = (a0 + m * TEAM) % NS * (LEN / (NS * R));
            bool turn = m * TEAM + TEAM > U.lo && m * TEAM < U.hi;
            if (turn && (m * TEAM < U.lo || m * TEAM + TEAM > U.hi)) {
                // a wavefront's rows (8 at most, lo and hi being multiples of 16) are on one side
                const int j = __builtin_amdgcn_readfirstlane(a0) + m * TEAM;
                turn = j >= U.lo && j < U.hi;
            }
#pragma unroll
            for (int r = 1; r < R; ++r) x[r] = cmul(x[r], tw[r * k], turn && !last);
        }
        dft<T, R>(x);
#pragma unroll
        for (int r = 0; r < R; ++r) v[m + r * BPT] = x[r];
    }
}

// The stages that follow transforms of length NS, on rows a0 + q TEAM of a line and
// back to them.  A stage's result r of butterfly j belongs to row (j / NS) NS R + j %
// NS + r NS: in this thread when TEAM divides NS, otherwise it changes hands through
// LDS.  Adjacent lanes hold adjacent lines there (LP apart, odd), whatever the
// stage's stride: no two of 32 meet in a bank.
template <typename T, int LEN, int TEAM, bool FIRST, int NS>
__device__ __forceinline__ void line_stages(cplx<T>* v, cplx<T>* line, const cplx<T>* tw, int a0, bool last) {
    if constexpr (NS < LEN) {
        constexpr int R = Radix<LEN / NS>::value;
        constexpr int BPT = LEN / R / TEAM, PER = LEN / TEAM;
        butterflies<T, LEN, TEAM, FIRST, R, NS>(v, tw, a0, last);
        if constexpr (NS * R == LEN) {
            // rows j + r LEN / R: as they are
        } else if constexpr (NS % TEAM == 0) {
            cplx<T> u[PER];
#pragma unroll
            for (int m = 0; m < BPT; ++m) {
                constexpr int S = NS / TEAM;   // j / NS = m / S, j % NS = a0 + (m % S) TEAM
#pragma unroll
                for (int r = 0; r < R; ++r) u[m / S * (S * R) + m % S + r * S] = v[m + r * BPT];
            }
#pragma unroll
            for (int q = 0; q < PER; ++q) v[q] = u[q];
        } else {
            if constexpr (NS > 1) lds_barrier();   // the last exchange is read
#pragma unroll
            for (int m = 0; m < BPT; ++m) {
                const int j = a0 + m * TEAM;
                const int base = (j / NS) * (NS * R) + j % NS;
#pragma unroll
                for (int r = 0; r < R; ++r) line[base + r * NS] = v[m + r * BPT];
            }
            lds_barrier();
#pragma unroll
            for (int q = 0; q < PER; ++q) v[q] = line[a0 + q * TEAM];
        }
        line_stages<T, LEN, TEAM, FIRST, NS * R>(v, line, tw, a0, last);
    }
}

// Passes A and B.  Element (c, a, other, k2) of the [C][..][..][H] input sits
// at c*sComp + a*sAxis + other*sOther + k2 (output: the same with the
// output strides); the FFT runs along a.
// FIRST: input is the caller's spectrum (InT pairs), multiplied by the FP64
// symbol cAxis[a] * cOther[other] * c2[k2]; otherwise in-place on the work
// buffer (in == out).
template <typename T>
struct AxisArgs {
    const void* in;
    cplx<T>* out;
    int H, gx, gy;
    long sAxis, sOther, sComp, oAxis, oOther, oComp;
    const double *cAxis, *cOther, *c2;
    const cplx<T>* twg;
    int quarter;
};

// A workgroup's lines are W adjacent columns of one `other`, gx such blocks for the
// H columns.  What bounds it is HBM: 512^3 x 3 from a complex128 spectrum moves 4.9 GB
// at 4.6 TB/s (a copy reaches 5.2).  With the lines in LDS through all stages and one
// workgroup a CU the first pass took 1137 us and 52 for a launch of its own for the
// last column (1056 in this form), 1024^3 from complex64 3667 + 92 (2668); passes B
// 742 and 1988 (729, 1963).  32 lines of 512 points and one workgroup a CU took
// 1066, real and imaginary parts exchanged in turn for twice the lines 1400 (their
// registers spill).
template <typename T, typename InT, int LEN, bool FIRST>
__global__ __launch_bounds__((StridedCfg<T, LEN>::THREADS))
__attribute__((amdgpu_waves_per_eu(StridedCfg<T, LEN>::WAVES))) void
k_fft_axis(AxisArgs<T> g) {
    using Cfg = StridedCfg<T, LEN>;
    constexpr int W = Cfg::W, TEAM = Cfg::TEAM, PER = Cfg::PER;
    __shared__ cplx<T> lines[W * Cfg::LP];
    __shared__ cplx<T> tw[LEN];
    const int tid = threadIdx.x;
    const int w = tid % W, a0 = tid / W;   // rows a0 + q TEAM of line w
    int lb = blockIdx.x;
    if constexpr (FIRST) {
        // Workgroups are dispatched round-robin over the 8 XCDs; here each XCD is
        // given one contiguous range of logical blocks instead, so that the
        // column blocks of one row set run on one XCD and the cache lines they
        // share in the caller's (unaligned) rows are L2 hits.  The work
        // buffer's rows are aligned, and the plain order measured as fast or
        // faster there.
        const int q8 = gridDim.x / 8, r8 = gridDim.x % 8, x8 = lb % 8;
        lb = x8 * q8 + (x8 < r8 ? x8 : r8) + lb / 8;
    }
    const int other = lb / g.gx % g.gy, bz = lb / (g.gx * g.gy);
    const int k2_0 = lb % g.gx * W;
    const bool valid = k2_0 + w < g.H;
    const int k2 = k2_0 + (valid ? w : 0);
    const long lane_base = long(bz) * g.sComp + long(other) * g.sOther + k2 + long(a0) * g.sAxis;
    const long step = long(TEAM) * g.sAxis;
    const long olane_base = long(bz) * g.oComp + long(other) * g.oOther + k2 + long(a0) * g.oAxis;
    const long ostep = long(TEAM) * g.oAxis;
    cplx<T> v[PER];
    if constexpr (FIRST) {
        const InT* in = static_cast<const InT*>(g.in);
        const double cw = g.c2[k2];
        const double cO = g.cOther[other];
        InT re[PER], im[PER];
        double ca[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const long e = lane_base + q * step;
            re[q] = in[2 * e];
            im[q] = in[2 * e + 1];
            ca[q] = g.cAxis[q * TEAM + a0];
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const double m = (ca[q] * cO) * cw;
            const double a = double(re[q]) * m, b = double(im[q]) * m;
            // times i^quarter (the i's of derivative factors; 0 otherwise)
            const double x = g.quarter == 0 ? a : g.quarter == 1 ? -b : g.quarter == 2 ? -a : b;
            const double y = g.quarter == 0 ? b : g.quarter == 1 ? a : g.quarter == 2 ? -b : -a;
            v[q] = {T(x), T(y)};
        }
    } else {
        const cplx<T>* src = static_cast<const cplx<T>*>(g.in);
#pragma unroll
        for (int q = 0; q < PER; ++q) v[q] = src[lane_base + q * step];
    }
    for (int i = tid; i < LEN; i += Cfg::THREADS) tw[i] = g.twg[i];
    cplx<T>* line = lines + w * Cfg::LP;
    constexpr int ALONE = LEN < 1024 ? 32 : sizeof(T) == 4 ? 16 : 8;
    const bool last = FIRST && LEN >= 256 && k2_0 > 0 && k2_0 == g.H - 1 && k2_0 % ALONE == 0;
    // tw is read after the barrier of the stages' first exchange; a line on one thread
    // (12 and 24 points) exchanges nothing
    if constexpr (TEAM == 1) lds_barrier();
    line_stages<T, LEN, TEAM, FIRST, 1>(v, line, tw, a0, last);
    if (valid) {
#pragma unroll
        for (int q = 0; q < PER; ++q) g.out[olane_base + q * ostep] = v[q];
    }
}

// ---- storage conversions -------------------------------------------------

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    // IEEE binary32 -> bfloat16, round to nearest, ties to even; NaN stays NaN.
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}
template <typename O, typename T>
__device__ __forceinline__ O store_cast(T v) {
    if constexpr (sizeof(O) == 2) return f32_to_bf16_rne(float(v));
    else return O(v);
}
template <typename O>
__device__ __forceinline__ double load_widen(O v) {
    if constexpr (sizeof(O) == 2) return double(__uint_as_float(uint32_t(v) << 16));
    else return double(v);
}

// Pass C configuration: TEAM threads per length-M transform, LINES grid rows of
// C components per workgroup.
template <typename T, int M, int C>
struct C2rCfg {
    static constexpr int TEAM = M >= 512 ? 64 : M >= 256 ? 32 : M >= 128 ? 16 : 8;
    static constexpr int LINES0 = 256 / (C * TEAM);
    // keep the LDS rows (plus the 2M twiddles) within about 40 KB
    static constexpr int LP = spread_len<T>(M + 2);
    static constexpr int LBYTES = (40 * 1024 - 2 * M * int(sizeof(cplx<T>))) / (C * LP * int(sizeof(cplx<T>)));
    static constexpr int LINES1 = LINES0 < LBYTES ? LINES0 : LBYTES;
    static constexpr int LINES = LINES1 < 1 ? 1 : LINES1;
    static constexpr int THREADS = LINES * C * TEAM;
};

// Pieces of pass C.  A workgroup holds NL lines of M + 1 half-spectrum values in
// zb, LP apart (M + 2, FP64 ones spread), with the twiddles tw[m] = exp(+2 pi i m / (2M)), m < 2M.

// The lines from work[c][g0][g1][k2] (rows of Hp, at least M + 2): line l of the
// block is zb line l * C + c.  All loads of a thread are issued before its stores;
// 16 bytes each (the last pair of FP32 values ends in the row's padding).
template <typename T, int M, int C, int LINES, int THREADS>
__device__ __forceinline__ void c2r_load(const cplx<T>* __restrict__ work, int Hp, long nlines, cplx<T>* zb) {
    constexpr int LP = spread_len<T>(M + 2), NL = LINES * C;
    constexpr int VEC = 16 / int(sizeof(cplx<T>));      // values per load
    constexpr int NV = (M + 1 + VEC - 1) / VEC;         // loads per line
    constexpr int ITER = (NL * NV + THREADS - 1) / THREADS;
    const long line0 = long(blockIdx.x) * LINES;
    const long compStride = nlines * Hp;
    u32x4 v[ITER];
#pragma unroll
    for (int q = 0; q < ITER; ++q) {
        const int idx = q * THREADS + int(threadIdx.x);
        const int f = idx / NV, k = idx - f * NV;
        const int l = f / C, c = f - l * C;
        const bool ok = idx < NL * NV && line0 + l < nlines;
        v[q] = *reinterpret_cast<const u32x4*>(work + (ok ? long(c) * compStride + (line0 + l) * Hp + k * VEC : 0));
    }
#pragma unroll
    for (int q = 0; q < ITER; ++q) {
        const int idx = q * THREADS + int(threadIdx.x);
        union {
            u32x4 v;
            cplx<T> z[VEC];
        } o;
        o.v = v[q];
        if (idx < NL * NV) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) zb[idx / NV * LP + spread<T>(idx % NV * VEC + i)] = o.z[i];
        }
    }
}

// Even/odd twist of NL lines: Z[k] = (X[k] + conj X[M-k]) + i e^{2 pi i k/(2M)}
// (X[k] - conj X[M-k]), with the imaginary parts of X[0] and X[M] dropped
// (real-FFT semantics).  After the length-M transform, real value g of the line is
// word real_word(g).
template <typename T>
__device__ __forceinline__ int real_word(int g) { return 2 * spread<T>(g >> 1) + (g & 1); }
template <typename T, int M, int NL, int THREADS>
__device__ __forceinline__ void c2r_twist(cplx<T>* zb, const cplx<T>* tw) {
    constexpr int LP = spread_len<T>(M + 2);
    for (int idx = threadIdx.x; idx < NL * (M / 2 + 1); idx += THREADS) {
        const int f = idx / (M / 2 + 1), k = idx % (M / 2 + 1);
        cplx<T>* X = zb + f * LP;
        if (k == 0) {
            const T a = X[0].x, b = X[spread<T>(M)].x;
            X[0] = {a + b, a - b};
        } else {
            const int kk = M - k;
            const cplx<T> A = X[spread<T>(k)], B = X[spread<T>(kk)];
            const cplx<T> Bc = {B.x, -B.y}, Ac = {A.x, -A.y};
            const cplx<T> z1 = cadd(cadd(A, Bc), cmul_i(cmul(csub(A, Bc), tw[k])));
            if (k < kk) {
                const cplx<T> z2 = cadd(cadd(B, Ac), cmul_i(cmul(csub(B, Ac), tw[kk])));
                X[spread<T>(kk)] = z2;
            }
            X[spread<T>(k)] = z1;
        }
    }
}

// The padded grid rows that a line goes to: itself and its periodic ghost copies.
// Grid point g of axes 0 and 1 stands at p(g) = st g + o; one copy minus or plus
// st n where that is inside [0, P).
struct RowTargets {
    long at[4];   // element offsets; -1: none
};
__device__ __forceinline__ RowTargets row_targets(long line, int n0, int n1, int P0, int P1, int pitch2, int st,
                                                  int o0, int o1) {
    const int g0 = int(line / n1), g1 = int(line % n1);
    const int p0a = st * g0 + o0, p1a = st * g1 + o1;
    const int p0b = p0a - st * n0 >= 0 ? p0a - st * n0 : p0a + st * n0 < P0 ? p0a + st * n0 : -1;
    const int p1b = p1a - st * n1 >= 0 ? p1a - st * n1 : p1a + st * n1 < P1 ? p1a + st * n1 : -1;
    RowTargets r;
    r.at[0] = (long(p0a) * P1 + p1a) * pitch2;
    r.at[1] = p1b >= 0 ? (long(p0a) * P1 + p1b) * pitch2 : -1;
    r.at[2] = p0b >= 0 ? (long(p0b) * P1 + p1a) * pitch2 : -1;
    r.at[3] = p0b >= 0 && p1b >= 0 ? (long(p0b) * P1 + p1b) * pitch2 : -1;
    return r;
}

// Writes the rows of the block's lines, 16 bytes a thread, the chunks of all lines
// dealt to the threads together (a row has as few as 35 values).  value(l, e) is
// element e < rowElems of line l; the row's padding is written as zeros.
template <typename OutT, int LINES, int THREADS, typename ValueFn>
__device__ __forceinline__ void c2r_store(OutT* __restrict__ grid, const RowTargets* rows, int lines, int rowElems,
                                          ValueFn value) {
    constexpr int VEC = 16 / int(sizeof(OutT));
    const int chunks = (rowElems + VEC - 1) / VEC;
    // idx / chunks for idx < 2^22: the quotient of the midpoints is at least 1 / (2
    // chunks) away from the next integer
    const float inv = 1.0f / float(chunks);
    for (int idx = threadIdx.x; idx < lines * chunks; idx += THREADS) {
        const int l = LINES == 1 ? 0 : int((float(idx) + 0.5f) * inv);
        const int e0 = (idx - l * chunks) * VEC;
        union {
            u32x4 v;
            OutT e[VEC];
        } o;
#pragma unroll
        for (int i = 0; i < VEC; ++i) o.e[i] = e0 + i < rowElems ? value(l, e0 + i) : OutT(0);
        const RowTargets& r = rows[l];
        *reinterpret_cast<u32x4*>(grid + r.at[0] + e0) = o.v;
#pragma unroll
        for (int j = 1; j < 4; ++j)
            if (r.at[j] >= 0) *reinterpret_cast<u32x4*>(grid + r.at[j] + e0) = o.v;
    }
}

// Pass C.  work[c][g0][g1][k2] (k2 <= M, rows of Hp) -> grid[p0][p1][p2][c] with ghost
// planes: padded index p holds grid index (p - padlo) mod n on every axis.
template <typename T, typename OutT, int M, int C>
__global__ __launch_bounds__(256) void k_c2r(const cplx<T>* __restrict__ work, int Hp, OutT* __restrict__ grid,
                                             int n0, int n1, int P0, int P1, int P2, int pitch2,
                                             int padlo, const cplx<T>* __restrict__ twg) {
    using Cfg = C2rCfg<T, M, C>;
    constexpr int LP = Cfg::LP;
    constexpr int NL = Cfg::LINES * C;  // transforms per block
    __shared__ __align__(16) cplx<T> zb[NL * LP];
    __shared__ cplx<T> tw[2 * M];
    __shared__ RowTargets rows[Cfg::LINES];
    const int tid = threadIdx.x;
    const long nlines = long(n0) * n1;
    const long line0 = long(blockIdx.x) * Cfg::LINES;
    const int lines = int(min(long(Cfg::LINES), nlines - line0));

    for (int i = tid; i < 2 * M; i += Cfg::THREADS) tw[i] = twg[i];
    if (tid < lines) rows[tid] = row_targets(line0 + tid, n0, n1, P0, P1, pitch2, 1, padlo, padlo);
    c2r_load<T, M, C, Cfg::LINES, Cfg::THREADS>(work, Hp, nlines, zb);
    lds_barrier();
    c2r_twist<T, M, NL, Cfg::THREADS>(zb, tw);
    lds_barrier();
    fft_stages<T, M, Cfg::TEAM, 1, 2>(zb + (tid / Cfg::TEAM) * LP, tw, tid % Cfg::TEAM);
    const T* real = reinterpret_cast<const T*>(zb);
    c2r_store<OutT, Cfg::LINES, Cfg::THREADS>(grid, rows, lines, P2 * C, [&](int l, int e) {
        const int p2 = e / C, c = e % C;
        int g2 = p2 - padlo;
        g2 += g2 < 0 ? 2 * M : g2 >= 2 * M ? -2 * M : 0;
        return store_cast<OutT>(real[(l * C + c) * 2 * LP + real_word<T>(g2)]);
    });
}

// Pass C of a Hermite field pair: from one line X of the half spectrum (the
// axis-0/1 derivative factors already applied) the fields with axis-2
// derivative order 0 and 1 -- Y[k] = i d[k] X[k], d the derivative table of
// axis 2 -- each by the even/odd twist and a length-M FFT, written together:
// doubled grid entry 2 g + a2 (+ the offsets a0, a1 of axes 0 and 1) holds
// field a2 at grid point g, so whole rows are written.  dtab[k] = 2 pi k / n2
// for k < M, 0 at the Nyquist index M.
// (Three components of 1024 points take six teams of 64 threads.)
template <typename T, typename OutT, int M, int C>
__global__ __launch_bounds__((C2rCfg<T, M, 2 * C>::THREADS > 256 ? C2rCfg<T, M, 2 * C>::THREADS : 256)) void
k_c2r_dual(const cplx<T>* __restrict__ work, int Hp, OutT* __restrict__ grid, int n0, int n1, int P0, int P1, int P2,
                                                  int pitch2, const cplx<T>* __restrict__ twg,
                                                  const double* __restrict__ dtab, int a0, int a1) {
    using Cfg = C2rCfg<T, M, 2 * C>;
    constexpr int H = M + 1;
    constexpr int LP = Cfg::LP;
    constexpr int NL = Cfg::LINES * C;  // lines of X per block; the Y lines follow
    __shared__ __align__(16) cplx<T> zb[2 * NL * LP];
    __shared__ cplx<T> tw[2 * M];
    __shared__ RowTargets rows[Cfg::LINES];
    const int tid = threadIdx.x;
    const long nlines = long(n0) * n1;
    const long line0 = long(blockIdx.x) * Cfg::LINES;
    const int lines = int(min(long(Cfg::LINES), nlines - line0));

    for (int i = tid; i < 2 * M; i += Cfg::THREADS) tw[i] = twg[i];
    if (tid < lines) rows[tid] = row_targets(line0 + tid, n0, n1, P0, P1, pitch2, 2, a0, a1);
    c2r_load<T, M, C, Cfg::LINES, Cfg::THREADS>(work, Hp, nlines, zb);
    lds_barrier();
    for (int idx = tid; idx < NL * H; idx += Cfg::THREADS) {
        const int f = idx / H, k = idx - f * H;
        const T d = T(dtab[k]);
        const cplx<T> x = zb[f * LP + spread<T>(k)];
        zb[(NL + f) * LP + spread<T>(k)] = {-d * x.y, d * x.x};  // i d X
    }
    lds_barrier();
    c2r_twist<T, M, 2 * NL, Cfg::THREADS>(zb, tw);
    lds_barrier();
    fft_stages<T, M, Cfg::TEAM, 1, 2>(zb + (tid / Cfg::TEAM) * LP, tw, tid % Cfg::TEAM);
    // rows of the doubled grid: both parities of axis 2
    const T* real = reinterpret_cast<const T*>(zb);
    c2r_store<OutT, Cfg::LINES, Cfg::THREADS>(grid, rows, lines, P2 * C, [&](int l, int e) {
        const int p2 = e / C, c = e % C;
        int g2 = p2 >> 1;
        if (g2 >= 2 * M) g2 -= 2 * M;
        return store_cast<OutT>(real[((p2 & 1 ? NL : 0) + l * C + c) * 2 * LP + real_word<T>(g2)]);
    });
}

// Dense FP64 [C][n0][n1][n2] <-> padded interleaved grid.
template <typename O>
__global__ void k_from_dense(const double* __restrict__ dense, O* __restrict__ grid, int C, int n0,
                             int n1, int n2, int P0, int P1, int P2, int pitch2, int padlo) {
    const long total = long(P0) * P1 * P2 * C;
    for (long i = blockIdx.x * long(blockDim.x) + threadIdx.x; i < total;
         i += long(gridDim.x) * blockDim.x) {
        const int c = int(i % C);
        long r = i / C;
        const int p2 = int(r % P2);
        r /= P2;
        const int p1 = int(r % P1);
        const int p0 = int(r / P1);
        int g0 = p0 - padlo, g1 = p1 - padlo, g2 = p2 - padlo;
        g0 += (g0 < 0) ? n0 : (g0 >= n0 ? -n0 : 0);
        g1 += (g1 < 0) ? n1 : (g1 >= n1 ? -n1 : 0);
        g2 += (g2 < 0) ? n2 : (g2 >= n2 ? -n2 : 0);
        grid[(long(p0) * P1 + p1) * pitch2 + long(p2) * C + c] =
            store_cast<O>(dense[((long(c) * n0 + g0) * n1 + g1) * n2 + g2]);
    }
}
template <typename O>
__global__ void k_to_dense(const O* __restrict__ grid, double* __restrict__ dense, int C, int n0,
                           int n1, int n2, int P1, int pitch2, int padlo) {
    const long total = long(C) * n0 * n1 * n2;
    for (long i = blockIdx.x * long(blockDim.x) + threadIdx.x; i < total;
         i += long(gridDim.x) * blockDim.x) {
        long r = i;
        const int g2 = int(r % n2);
        r /= n2;
        const int g1 = int(r % n1);
        r /= n1;
        const int g0 = int(r % n0);
        const int c = int(r / n0);
        dense[i] = load_widen<O>(
            grid[(long(g0 + padlo) * P1 + (g1 + padlo)) * pitch2 + long(g2 + padlo) * C + c]);
    }
}

// ------------------------------------------------------------- launchers ---

namespace {

template <typename T, typename InT, bool FIRST>
bsi_status launch_axis(int len, int others, int C, const InT* in, cplx<T>* out, int H, long sAxis, long sOther,
                       long sComp, long oAxis, long oOther, long oComp, const double* cAxis,
                       const double* cOther, const double* c2, const cplx<T>* tw, hipStream_t s, int quarter = 0) {
#define BSI_AXIS_CASE(L)                                                                           \
    case L: {                                                                                      \
        using Cfg = StridedCfg<T, L>;                                                              \
        const int gx = (H + Cfg::W - 1) / Cfg::W;                                                  \
        hipLaunchKernelGGL((k_fft_axis<T, InT, L, FIRST>), dim3(unsigned(gx) * unsigned(others * C)), \
                           dim3(Cfg::THREADS), 0, s,                                               \
                           AxisArgs<T>{in, out, H, gx, others, sAxis, sOther, sComp, oAxis, oOther, oComp, cAxis, \
                                       cOther, c2, tw, quarter});                                  \
        break;                                                                                     \
    }
    switch (len) {
        BSI_AXIS_CASE(8)
        BSI_AXIS_CASE(12)
        BSI_AXIS_CASE(16)
        BSI_AXIS_CASE(24)
        BSI_AXIS_CASE(32)
        BSI_AXIS_CASE(48)
        BSI_AXIS_CASE(64)
        BSI_AXIS_CASE(96)
        BSI_AXIS_CASE(128)
        BSI_AXIS_CASE(192)
        BSI_AXIS_CASE(256)
        BSI_AXIS_CASE(384)
        BSI_AXIS_CASE(512)
        BSI_AXIS_CASE(768)
        BSI_AXIS_CASE(1024)
        default:
            set_error("unsupported FFT length " + std::to_string(len));
            return BSI_E_UNSUPPORTED;
    }
#undef BSI_AXIS_CASE
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

template <typename T, typename OutT, int C>
bsi_status launch_c2r(int M, const cplx<T>* work, int Hp, OutT* grid, int n0, int n1, int P0, int P1, int P2,
                      int pitch2, int padlo, const cplx<T>* tw, hipStream_t s) {
    const long nlines = long(n0) * n1;
#define BSI_C2R_CASE(MM)                                                                           \
    case MM: {                                                                                     \
        using Cfg = C2rCfg<T, MM, C>;                                                                 \
        const unsigned nb = unsigned((nlines + Cfg::LINES - 1) / Cfg::LINES);                      \
        hipLaunchKernelGGL((k_c2r<T, OutT, MM, C>), dim3(nb), dim3(Cfg::THREADS), 0, s, work, Hp, grid, \
                           n0, n1, P0, P1, P2, pitch2, padlo, tw);                                \
        break;                                                                                     \
    }
    switch (M) {
        BSI_C2R_CASE(4)
        BSI_C2R_CASE(6)
        BSI_C2R_CASE(8)
        BSI_C2R_CASE(12)
        BSI_C2R_CASE(16)
        BSI_C2R_CASE(24)
        BSI_C2R_CASE(32)
        BSI_C2R_CASE(48)
        BSI_C2R_CASE(64)
        BSI_C2R_CASE(96)
        BSI_C2R_CASE(128)
        BSI_C2R_CASE(192)
        BSI_C2R_CASE(256)
        BSI_C2R_CASE(384)
        BSI_C2R_CASE(512)
        default:
            set_error("unsupported real FFT length " + std::to_string(2 * M));
            return BSI_E_UNSUPPORTED;
    }
#undef BSI_C2R_CASE
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

template <typename T, typename OutT, int C>
bsi_status launch_c2r_dual(int M, const cplx<T>* work, int Hp, OutT* grid, int n0, int n1, int P0, int P1,
                           int P2, int pitch2, const cplx<T>* tw, const double* dtab, int a0, int a1,
                           hipStream_t s) {
    const long nlines = long(n0) * n1;
#define BSI_C2RD_CASE(MM)                                                                          \
    case MM: {                                                                                     \
        using Cfg = C2rCfg<T, MM, 2 * C>;                                                          \
        const unsigned nb = unsigned((nlines + Cfg::LINES - 1) / Cfg::LINES);                      \
        hipLaunchKernelGGL((k_c2r_dual<T, OutT, MM, C>), dim3(nb), dim3(Cfg::THREADS), 0, s, work, Hp, grid, \
                           n0, n1, P0, P1, P2, pitch2, tw, dtab, a0, a1);                          \
        break;                                                                                     \
    }
    switch (M) {
        BSI_C2RD_CASE(4)
        BSI_C2RD_CASE(6)
        BSI_C2RD_CASE(8)
        BSI_C2RD_CASE(12)
        BSI_C2RD_CASE(16)
        BSI_C2RD_CASE(24)
        BSI_C2RD_CASE(32)
        BSI_C2RD_CASE(48)
        BSI_C2RD_CASE(64)
        BSI_C2RD_CASE(96)
        BSI_C2RD_CASE(128)
        BSI_C2RD_CASE(192)
        BSI_C2RD_CASE(256)
        BSI_C2RD_CASE(384)
        BSI_C2RD_CASE(512)
        default:
            set_error("unsupported real FFT length " + std::to_string(2 * M));
            return BSI_E_UNSUPPORTED;
    }
#undef BSI_C2RD_CASE
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

template <typename T, typename InT, typename OutT>
bsi_status prefilter_pass(bsi_field* f, const InT* uhat, OutT* grid, cplx<T>* work, int H, int Hp, long sComp,
                          long wComp, const double* const* ct, const int* a, int quarter,
                          const void* tw0, const void* tw1, const void* tw2, hipStream_t s,
                          const double* dual_tab = nullptr);

template <typename T, typename InT, typename OutT>
bsi_status prefilter_typed(bsi_field* f, const InT* uhat, OutT* grid, hipStream_t s) {
    bsi_ctx* ctx = f->ctx;
    const int n0 = f->n[0], n1 = f->n[1], n2 = f->n[2], C = f->C;
    const int H = n2 / 2 + 1;
    // work rows padded to whole 128-byte lines, so that the W-column row
    // segments of the strided passes do not straddle an extra line
    constexpr int LINE = 128 / int(sizeof(cplx<T>));
    const int Hp = (H + LINE - 1) / LINE * LINE;
    const size_t elems = size_t(C) * n0 * n1 * Hp;
    void* wsp = nullptr;
    BSI_TRY(get_workspace(ctx->fft_ws, s, elems * sizeof(cplx<T>), &wsp));
    cplx<T>* work = static_cast<cplx<T>*>(wsp);
    const void *tw0, *tw1, *tw2;
    const bool dbl = sizeof(T) == 8;
    BSI_TRY(get_twiddles(ctx, n0, dbl, &tw0));
    BSI_TRY(get_twiddles(ctx, n1, dbl, &tw1));
    BSI_TRY(get_twiddles(ctx, n2, dbl, &tw2));
    const long sComp = long(n0) * n1 * H;    // caller's spectrum
    const long wComp = long(n0) * n1 * Hp;   // work buffer
    // one inverse FFT per stored field: the prefiltered (or plain) field, or
    // for Hermite the 8 derivative fields d^(a0+a1+a2) u / ds0^a0 ds1^a1 ds2^a2,
    // where the two fields of each (a0, a1) share the axis-0 and axis-1 passes
    // and one pass C writes both (k_c2r_dual)
    const bool herm = f->basis == BSI_BASIS_HERMITE;
    const int nn[3] = {n0, n1, n2};
    if (!herm) {
        const int a[3] = {0, 0, 0};
        const double* ct[3];
        for (int d = 0; d < 3; ++d) BSI_TRY(get_ctable(ctx, nn[d], f->N, f->desc.prefilter, &ct[d]));
        return prefilter_pass<T, InT, OutT>(f, uhat, grid, work, H, Hp, sComp, wComp, ct, a, 0, tw0, tw1, tw2,
                                            s);
    }
    const double* dtab2 = nullptr;
    BSI_TRY(get_ctable(ctx, n2, f->N, DERIVATIVE_TABLE, &dtab2));
    for (int pr = 0; pr < 4; ++pr) {
        const int a[3] = {(pr >> 1) & 1, pr & 1, 0};
        const double* ct[3];
        for (int d = 0; d < 2; ++d)
            BSI_TRY(get_ctable(ctx, nn[d], f->N, a[d] ? DERIVATIVE_TABLE : BSI_PREFILTER_NONE, &ct[d]));
        BSI_TRY(get_ctable(ctx, n2, f->N, BSI_PREFILTER_NONE, &ct[2]));
        BSI_TRY((prefilter_pass<T, InT, OutT>(f, uhat, grid, work, H, Hp, sComp, wComp, ct, a,
                                              (a[0] + a[1]) & 3, tw0, tw1, tw2, s, dtab2)));
    }
    return BSI_OK;
}

// The three passes of one inverse FFT: symbol tables ct[d] per axis, the
// product times i^quarter; with dual_tab, pass C writes the Hermite pair of axis-2
// orders 0 and 1 at offsets a[0], a[1] (k_c2r_dual, dual_tab the axis-2 derivative
// table).
template <typename T, typename InT, typename OutT>
bsi_status prefilter_pass(bsi_field* f, const InT* uhat, OutT* grid, cplx<T>* work, int H, int Hp, long sComp,
                          long wComp, const double* const* ct, const int* a, int quarter,
                          const void* tw0, const void* tw1, const void* tw2, hipStream_t s,
                          const double* dual_tab) {
    bsi_ctx* ctx = f->ctx;
    const int n0 = f->n[0], n1 = f->n[1], n2 = f->n[2], C = f->C;
    const double *c0 = ct[0], *c1 = ct[1], *c2 = ct[2];
    // pass A: axis 0 (stride n1*H in, n1*Hp out), other = k1 (stride H in, Hp out)
    {
    StageTimer tm(ctx, "fft_axis0", s);
    BSI_TRY((launch_axis<T, InT, true>(n0, n1, C, uhat, work, H, long(n1) * H, long(H), sComp,
                                       long(n1) * Hp, long(Hp), wComp, c0, c1, c2,
                                       static_cast<const cplx<T>*>(tw0), s, quarter)));
    }
    // pass B: axis 1 (stride Hp), other = k0 (stride n1*Hp), in place
    {
    StageTimer tm(ctx, "fft_axis1", s);
    BSI_TRY((launch_axis<T, T, false>(n1, n0, C, reinterpret_cast<const T*>(work), work, H,
                                      long(Hp), long(n1) * Hp, wComp, long(Hp), long(n1) * Hp, wComp, nullptr,
                                      nullptr, nullptr, static_cast<const cplx<T>*>(tw1), s)));
    }
    // pass C: c2r along axis 2
    const int M = n2 / 2;
    StageTimer tm(ctx, "fft_c2r", s);
    if (dual_tab) {
        const cplx<T>* t2 = static_cast<const cplx<T>*>(tw2);
        if (C == 1)
            return launch_c2r_dual<T, OutT, 1>(M, work, Hp, grid, n0, n1, f->P[0], f->P[1], f->P[2], f->pitch2, t2,
                                               dual_tab, a[0], a[1], s);
        return launch_c2r_dual<T, OutT, 3>(M, work, Hp, grid, n0, n1, f->P[0], f->P[1], f->P[2], f->pitch2, t2,
                                           dual_tab, a[0], a[1], s);
    }
    if (C == 1)
        return launch_c2r<T, OutT, 1>(M, work, Hp, grid, n0, n1, f->P[0], f->P[1], f->P[2], f->pitch2, f->padlo,
                                      static_cast<const cplx<T>*>(tw2), s);
    return launch_c2r<T, OutT, 3>(M, work, Hp, grid, n0, n1, f->P[0], f->P[1], f->P[2], f->pitch2, f->padlo,
                                  static_cast<const cplx<T>*>(tw2), s);
}

}  // namespace

bsi_status prefilter_run(bsi_field* f, const void* uhat, int prec, hipStream_t s) {
    const int coef = f->desc.coef;
    if (coef == BSI_F64) {
        if (prec == BSI_F64)
            return prefilter_typed<double, double, double>(f, static_cast<const double*>(uhat),
                                                           static_cast<double*>(f->grid), s);
        return prefilter_typed<double, float, double>(f, static_cast<const float*>(uhat),
                                                      static_cast<double*>(f->grid), s);
    }
    if (coef == BSI_F32) {
        if (prec == BSI_F64)
            return prefilter_typed<float, double, float>(f, static_cast<const double*>(uhat),
                                                         static_cast<float*>(f->grid), s);
        return prefilter_typed<float, float, float>(f, static_cast<const float*>(uhat),
                                                    static_cast<float*>(f->grid), s);
    }
    if (prec == BSI_F64)
        return prefilter_typed<float, double, uint16_t>(f, static_cast<const double*>(uhat),
                                                        static_cast<uint16_t*>(f->grid), s);
    return prefilter_typed<float, float, uint16_t>(f, static_cast<const float*>(uhat),
                                                   static_cast<uint16_t*>(f->grid), s);
}

bsi_status grid_from_dense(bsi_field* f, const double* dense, hipStream_t s) {
    const long total = long(f->P[0]) * f->P[1] * f->P[2] * f->C;
    const unsigned nb = unsigned(std::min<long>((total + 255) / 256, 65535L * 8));
    if (f->desc.coef == BSI_F64)
        hipLaunchKernelGGL(k_from_dense<double>, dim3(nb), dim3(256), 0, s, dense,
                           static_cast<double*>(f->grid), f->C, f->gn[0], f->gn[1], f->gn[2], f->P[0],
                           f->P[1], f->P[2], f->pitch2, f->padlo);
    else if (f->desc.coef == BSI_F32)
        hipLaunchKernelGGL(k_from_dense<float>, dim3(nb), dim3(256), 0, s, dense,
                           static_cast<float*>(f->grid), f->C, f->gn[0], f->gn[1], f->gn[2], f->P[0],
                           f->P[1], f->P[2], f->pitch2, f->padlo);
    else
        hipLaunchKernelGGL(k_from_dense<uint16_t>, dim3(nb), dim3(256), 0, s, dense,
                           static_cast<uint16_t*>(f->grid), f->C, f->gn[0], f->gn[1], f->gn[2], f->P[0],
                           f->P[1], f->P[2], f->pitch2, f->padlo);
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

bsi_status grid_to_dense(const bsi_field* f, double* dense, hipStream_t s) {
    const long total = long(f->C) * f->gn[0] * f->gn[1] * f->gn[2];
    const unsigned nb = unsigned(std::min<long>((total + 255) / 256, 65535L * 8));
    if (f->desc.coef == BSI_F64)
        hipLaunchKernelGGL(k_to_dense<double>, dim3(nb), dim3(256), 0, s,
                           static_cast<const double*>(f->grid), dense, f->C, f->gn[0], f->gn[1], f->gn[2],
                           f->P[1], f->pitch2, f->padlo);
    else if (f->desc.coef == BSI_F32)
        hipLaunchKernelGGL(k_to_dense<float>, dim3(nb), dim3(256), 0, s,
                           static_cast<const float*>(f->grid), dense, f->C, f->gn[0], f->gn[1], f->gn[2],
                           f->P[1], f->pitch2, f->padlo);
    else
        hipLaunchKernelGGL(k_to_dense<uint16_t>, dim3(nb), dim3(256), 0, s,
                           static_cast<const uint16_t*>(f->grid), dense, f->C, f->gn[0], f->gn[1],
                           f->gn[2], f->P[1], f->pitch2, f->padlo);
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

}  // namespace bsi
