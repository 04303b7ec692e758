// Device-side building blocks of the evaluation shared by the single-field
// kernels (eval.hip) and the persistent multi-field kernel (batch.hip):
// position -> cell/offset, tile keys, the grouping by key, B-spline weights and the
// per-particle tensor contraction (Sections 2, 3, 5; Table 1).  Both callers
// run exactly these functions, so a particle's result does not depend on which
// kernel evaluated it.
#pragma once

#include <algorithm>
#include <utility>

#include "common.hpp"
#include "device.hpp"

namespace bsi {

// ---------------------------------------------------------- cell / offset ---
// Section 5 stencil rule in grid units: s = x * (n/L) as one FP64 product,
// f = floor(s), t = s - f, cell = f mod n (exact Euclidean remainder).
// Contraction is off so that s - f is not fused into an FMA with x * inv_h.
// Returns false when s is not finite.
__device__ __forceinline__ bool cell_of(double x, double inv_h, int n, int& cell, double& t) {
#pragma clang fp contract(off)
    const double s = x * inv_h;
    if (!isfinite(s)) return false;
    const double f = floor(s);
    t = s - f;
    if (f >= 0.0 && f < double(n)) {     // the usual case: x already in [0, L)
        cell = int(f);
        return true;
    }
    if (fabs(f) < 9007199254740992.0) {  // |f| < 2^53: exact in int64
        long long m = static_cast<long long>(f) % n;
        if (m < 0) m += n;
        cell = int(m);
    } else {                             // f = integer-valued double, fmod is exact
        double r = fmod(f, double(n));
        if (r < 0) r += double(n);
        cell = int(r);
    }
    return true;
}

struct CellArgs {
    const double* pos;
    long P;
    int n0, n1, n2;
    double ih0, ih1, ih2;
};

// ---------------------------------------------------------------- binning ---
// Particles are counting-sorted by the key (tile_key) of the tile (cell / T) that
// holds their cell; non-finite particles go to one extra bucket at the end.

__device__ __forceinline__ uint32_t spread3(uint32_t v) {  // 10 bits -> every third bit
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t compact3(uint32_t v) {  // inverse of spread3
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030c30c3u;
    v = (v | (v >> 4)) & 0x0300f00fu;
    v = (v | (v >> 8)) & 0x030000ffu;
    v = (v | (v >> 16)) & 0x000003ffu;
    return v;
}

static __global__ void k_fill_u32(uint32_t* p, long n, uint32_t v) {
    for (long i = blockIdx.x * long(blockDim.x) + threadIdx.x; i < n; i += long(gridDim.x) * blockDim.x)
        p[i] = v;
}

// Key of the tile with coordinates (a, b, c) in the evaluation's binning: bricks
// of 4^3 tiles in Morton order, in a brick four tiles along axis 0 in a row (a
// tiled gather slides its block from one to the next), the rows in 2D Morton order.
__device__ __forceinline__ uint32_t tile_key(uint32_t a, uint32_t b, uint32_t c) {
    const uint32_t brick = (spread3(a >> 2) << 2) | (spread3(b >> 2) << 1) | spread3(c >> 2);
    return (brick << 6) | ((b & 2u) << 4) | ((c & 2u) << 3) | ((b & 1u) << 3) | ((c & 1u) << 2) | (a & 3u);
}
// First cell of that tile (T cells an edge), packed as pack_cell does.
__device__ __forceinline__ uint32_t tile_origin(uint32_t key, uint32_t T) {
    const uint32_t brick = key >> 6;
    const uint32_t a = (compact3(brick >> 2) << 2) | (key & 3u);
    const uint32_t b = (compact3(brick >> 1) << 2) | ((key >> 4) & 2u) | ((key >> 3) & 1u);
    const uint32_t c = (compact3(brick) << 2) | ((key >> 3) & 2u) | ((key >> 2) & 1u);
    return (a * T << 20) | (b * T << 10) | (c * T);
}

// 16 bytes as a native vector (loads and stores of it are single instructions,
// never aggregate copies) and a load of it from global memory.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4 global_u32x4;

__device__ __forceinline__ u32x4 load_global16(const u32x4* p) {
    return *(global_u32x4*)p;
}

// ------------------------------------------------------- grouping by key ---
// Particles are grouped by bucket key with a two-level counting sort that uses
// no per-particle global atomics (their throughput, not the data volume, bounds
// a one-pass counting sort with one atomic per particle).  The keys [0, nbuckets) are
// split into `ncoarse` contiguous coarse ranges of at most GRP_FINE_MAX keys,
// sized by the caller so that each holds a few hundred particles:
//   k_grp_hist    each block of `ipt * GRP_BLOCK` grouping slots counts its
//                 particles per coarse range in LDS (counts stored block by
//                 block, so that they are written and read as whole rows)
//   k_grp_scan    exclusive scan of every range's counts over the blocks, and
//                 the ranges' totals
//   k_grp_coarse  each block scans the totals in LDS (its own copy: a launch
//                 of a single-block scan costs more than repeating it) and
//                 scatters its particles into the coarse ranges as 32-byte
//                 records; one more block cuts the ranges into spans
//                 (grp_span), and a span into chunks of GRP_CHUNK particles
//   k_grp_fine    one workgroup per span, independent of all others: the
//                 span's records are ranked by key in LDS and written in key
//                 order into the span's own slots, and its runs of equal keys
//                 become work items (cut into pieces of at most `ichunk`), dealt
//                 evenly to the span's chunks
// A range of more than a span has several, each sorted by itself: a bucket's
// particles then lie in several runs, each with items of its own.  Nothing reads
// buckets as wholes, so no table over all buckets is written, and a crowded
// range needs no exchange between its workgroups.  The order inside a run is
// whatever the LDS atomics give; no result depends on it.
// The blocks of the two coarse passes are mapped so that each XCD takes one
// contiguous range of slots, which keeps the partial-line writes of one coarse
// range in one L2.  What bounds it: memory (24 B of position read twice, a
// 32 B record written and read, 20 or 28 B written per particle) from about 10^7
// particles; the launches and their cache write-backs (about 5 us each) below.
//
// Loads of several slots are issued without a branch between them (a clamped
// index in the place of a skipped slot): with one, the compiler waits for each.
//
// KeySrc::fetch(i, slot) loads grouping slot i's particle (false: the slot
// holds none, the loaded one is some other) and KeySrc::place(slot, pl) finds its key, coarse range, cell and
// offset.  Coarse::range(c, &lo, &hi) gives the keys [lo, hi) of range c.

constexpr int GRP_BLOCK = 1024;
constexpr uint32_t GRP_FINE_MAX = 8192;      // keys per coarse range: 32 KB of LDS
constexpr uint32_t GRP_COARSE_MAX = 8193;    // coarse ranges (2^13, and one for the particles without a cell)
constexpr uint32_t GRP_CHUNK = 2048;         // particles per chunk
constexpr int GRP_FINE_BLOCK = 256;
constexpr int GRP_UNROLL = 4;                // slots per thread whose loads overlap in the coarse passes
constexpr long GRP_NBLK_MAX = 512;           // blocks of the coarse passes: two of 1024 threads per CU

// A particle on its way to its bucket, 32 bytes (two 16-byte vectors): key,
// index in its own position array, then either its FP64 position or (PACK)
// its FP32 offsets t in the cell and the packed cell.
struct alignas(16) GrpRec {
    uint32_t key, local;
    double x[3];
};
static_assert(sizeof(GrpRec) == 32, "grouping record is two 16-byte vectors");

// A particle's cell in one word (10 bits per axis: n <= 1024), or NO_CELL.
constexpr uint32_t NO_CELL = 0xffffffffu;
__device__ __forceinline__ uint32_t pack_cell(const int* c) {
    return (uint32_t(c[0]) << 20) | (uint32_t(c[1]) << 10) | uint32_t(c[2]);
}

// Where a particle belongs.
struct GrpPlace {
    uint32_t key, coarse;
    bool ok;        // false: no cell (the key is the bucket of such particles)
    int cell[3];
    double t[3];
};

__device__ __forceinline__ uint32_t grp_block(long nblk) {
    const long b = blockIdx.x;
    const long q = nblk / 8, r = nblk % 8;
    const long x = b % 8, i = b / 8;
    return uint32_t(x * q + (x < r ? x : r) + i);
}

// Exclusive scan of one value per thread over the workgroup (B threads); sh
// holds B / 64 words.  *total (may be the same for all) = the sum.
template <int B>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(incl, off, 64);
        if (lane >= off) incl += u;
    }
    if (lane == 63) sh[wid] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < B / 64; ++w) {
        const uint32_t u = sh[w];
        before += w < wid ? u : 0u;
        sum += u;
    }
    __syncthreads();
    *total = sum;
    return before + incl - v;
}

template <typename KeySrc>
static __global__ __launch_bounds__(GRP_BLOCK) void k_grp_hist(KeySrc ks, long nidx, int ipt, uint32_t ncoarse,
                                                              long nblk, uint32_t* __restrict__ counts,
                                                              uint32_t* __restrict__ ctl, int nctl) {
    extern __shared__ uint32_t lh[];
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nctl; i += GRP_BLOCK) ctl[i] = 0;
    for (uint32_t c = threadIdx.x; c < ncoarse; c += GRP_BLOCK) lh[c] = 0;
    __syncthreads();
    const uint32_t blk = grp_block(nblk);
    const long b0 = long(blk) * ipt * GRP_BLOCK;
    for (int q0 = 0; q0 < ipt; q0 += GRP_UNROLL) {
        typename KeySrc::Slot sl[GRP_UNROLL];
        bool have[GRP_UNROLL];
#pragma unroll
        for (int u = 0; u < GRP_UNROLL; ++u) {
            const long i = b0 + long(q0 + u) * GRP_BLOCK + threadIdx.x;
            have[u] = ks.fetch(min(i, nidx - 1), sl[u]) && q0 + u < ipt && i < nidx;
        }
#pragma unroll
        for (int u = 0; u < GRP_UNROLL; ++u) {
            if (!have[u]) continue;
            GrpPlace pl;
            ks.place(sl[u], pl);
            atomicAdd(&lh[pl.coarse], 1u);
        }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < ncoarse; c += GRP_BLOCK) counts[long(blk) * ncoarse + c] = lh[c];
}

// 64 ranges per workgroup, 16 groups of blocks: every range's counts become
// their exclusive scan over the blocks; total[c] = the range's particles.
static __global__ __launch_bounds__(1024) void k_grp_scan(uint32_t* __restrict__ counts, uint32_t nblk,
                                                         uint32_t ncoarse, uint32_t* __restrict__ total) {
    constexpr int GROUPS = 16, ROWS = int(GRP_NBLK_MAX) / GROUPS;
    __shared__ uint32_t part[GROUPS][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const uint32_t c = blockIdx.x * 64 + lane;
    const uint32_t rows = (nblk + GROUPS - 1) / GROUPS;   // at most ROWS
    const uint32_t r0 = g * rows;
    uint32_t v[ROWS];
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const bool ok = uint32_t(r) < rows && r0 + r < nblk && c < ncoarse;
        v[r] = ok ? counts[long(r0 + r) * ncoarse + c] : 0u;
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) sum += v[r];
    part[g][lane] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int w = 0; w < g; ++w) run += part[w][lane];
    if (c >= ncoarse) return;
    if (g == GROUPS - 1) total[c] = run + sum;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if (uint32_t(r) < rows && r0 + r < nblk) counts[long(r0 + r) * ncoarse + c] = run;
        run += v[r];
    }
}

// ---- work items -----------------------------------------------------------
// (first cell of the tile or NO_CELL, first binned slot, count, tag): a piece of a
// run of one bucket.
// A chunk's items stand together, in key order, at slots reserved for it by the
// chunk plan (descriptor word 3; the fine pass puts their count in word 2).
// The tiled gathers take them in units, equal parts of a chunk's items, so that
// no list of all items is needed: one kept in order costs another launch, one
// appended to by the chunks as they finish loses the order.
constexpr uint32_t ITEM_UNITS = 8192, ITEM_UNITS_BATCH = 32768;

// The chunks are split into ITEM_RANGES contiguous ranges, one per XCD
// (neighbouring tiles, whose blocks overlap, meet in the same L2); the next
// unit of range x is counted at ITEM_CTL_STRIDE * x, each counter on a 128-byte
// line of its own (atomics on one line serialise), then the counts of finished
// workgroups: of ITEM_GROUPS groups of workgroups, and of those groups.
constexpr int ITEM_RANGES = 8;
constexpr int ITEM_GROUPS = 32;
constexpr int ITEM_CTL_STRIDE = 32;
constexpr int ITEM_CTL_WORDS = ITEM_CTL_STRIDE * (ITEM_RANGES + ITEM_GROUPS + 1);

// First chunk of the x-th range of nch chunks.
__host__ __device__ inline uint32_t item_range_begin(uint32_t x, uint32_t nch) {
    return uint32_t(uint64_t(x) * nch / ITEM_RANGES);
}

// The items of a single evaluation.
struct OneField {
    bool items;
    uint32_t tile, nbuckets_finite;
    __device__ __forceinline__ bool wanted(uint32_t) const { return items; }
    __device__ __forceinline__ uint32_t origin(uint32_t, uint32_t key) const {
        return key == nbuckets_finite ? NO_CELL : tile_origin(key, tile);
    }
    __device__ __forceinline__ uint32_t tag(uint32_t) const { return 0; }
    // the chunk plan tells that the chunks of range c start at chunk g
    __device__ __forceinline__ void begin(uint32_t, uint32_t) const {}
    __device__ __forceinline__ void end(uint32_t) const {}
};

// Particles per span of a range of cnt particles over nf keys: a chunk where that is
// 128 particles a key on average, otherwise what a workgroup sorts in its registers
// or, where 128 a key (256 from two such spans on) take more, a longer span whose
// records are read twice.  Shorter runs cost the gather more than the sort saves.  With
// chunks sorted alone a crowded range's tiles lay in up to 16 runs (10^7 clustered
// particles at 512^3, order 6: gather FP32 1920 -> 1770 us, BF16 1525 -> 1435, binning
// 462 -> 492), and ranges of many keys in runs of a few particles (1024^3, 4 * 10^7:
// 8250 -> 4620, binning 2000 -> 2460).  Twice as many a key in ranges of less than 8192:
// 4 * 10^7 uniform at 512^3 binning 1962 -> 2113 and gather 5031 -> 5278.
constexpr uint32_t GRP_SPAN_REG = 4096;
constexpr uint32_t GRP_SPAN_MAX = 32768;
constexpr uint32_t GRP_SPAN_RUN = 128;
__host__ __device__ inline uint32_t grp_span(uint32_t nf, uint32_t cnt) {
    if (nf <= GRP_CHUNK / GRP_SPAN_RUN) return GRP_CHUNK;
    const uint32_t run = cnt > 2 * GRP_SPAN_REG ? 2 * GRP_SPAN_RUN : GRP_SPAN_RUN;
    const uint32_t n = (nf < GRP_SPAN_MAX / run ? nf : GRP_SPAN_MAX / run) * run;
    return n > GRP_SPAN_REG ? (n + GRP_CHUNK - 1) / GRP_CHUNK * GRP_CHUNK : GRP_SPAN_REG;
}

// Most items of a span of n particles over nf keys.
__host__ __device__ inline uint32_t grp_item_bound(uint32_t n, uint32_t nf, uint32_t ichunk) {
    return (n < nf ? n : nf) + n / ichunk;
}

// Chunk plan, by one workgroup of GRP_BLOCK threads: base[c] = first slot of
// range c (base[ncoarse] = all particles), desc[g] = (range, first slot,
// particles, first item slot) of chunk g, the chunks listed range by range.  The
// first chunk of a span stands for all of it, the others have GRP_FOLLOWS set; the
// fine pass gives each of them its part of the items (words 2 and 3).
// Thread t owns the ranges t * per ..
constexpr uint32_t GRP_FOLLOWS = 0x80000000u;
template <typename Coarse, typename Lists>
__device__ __forceinline__ void grp_plan_block(const Coarse& cm, const Lists& ls, const uint32_t* __restrict__ total,
                                               uint32_t ncoarse, uint32_t ichunk, uint32_t* __restrict__ base,
                                               u32x4* __restrict__ desc, uint32_t* __restrict__ nchunks,
                                               uint32_t* sh) {
    const uint32_t per = (ncoarse + GRP_BLOCK - 1) / GRP_BLOCK;
    const uint32_t c0 = threadIdx.x * per;
    uint32_t n = 0, m = 0, ib = 0;
    auto bound = [&](uint32_t c, uint32_t cnt) {
        uint32_t lo, hi;
        cm.range(c, lo, hi);
        const uint32_t span = grp_span(hi - lo, cnt), full = cnt / span, rem = cnt % span;
        return full * grp_item_bound(span, hi - lo, ichunk) + grp_item_bound(rem, hi - lo, ichunk);
    };
    for (uint32_t q = 0; q < per; ++q) {
        if (c0 + q >= ncoarse) break;
        const uint32_t cnt = total[c0 + q];
        n += cnt;
        m += (cnt + GRP_CHUNK - 1) / GRP_CHUNK;
        ib += bound(c0 + q, cnt);
    }
    uint32_t all, nch, dummy;
    uint32_t run = block_scan<GRP_BLOCK>(n, sh, &all);
    uint32_t g = block_scan<GRP_BLOCK>(m, sh, &nch);
    uint32_t slot = block_scan<GRP_BLOCK>(ib, sh, &dummy);
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t c = c0 + q;
        if (c >= ncoarse) break;
        const uint32_t cnt = total[c];
        base[c] = run;
        ls.begin(c, g);
        uint32_t lo, hi;
        cm.range(c, lo, hi);
        const uint32_t span = grp_span(hi - lo, cnt);
        for (uint32_t j = 0; j < cnt; j += span) {
            const uint32_t k = min(span, cnt - j);
            desc[g++] = u32x4{c, run + j, k, slot};
            for (uint32_t i = GRP_CHUNK; i < k; i += GRP_CHUNK) desc[g++] = u32x4{c | GRP_FOLLOWS, 0u, 0u, 0u};
            slot += grp_item_bound(k, hi - lo, ichunk);
        }
        run += cnt;
    }
    if (threadIdx.x == 0) {
        base[ncoarse] = all;
        *nchunks = nch;
        ls.end(nch);
    }
}

template <typename KeySrc, typename Coarse, typename Lists, bool PACK>
static __global__ __launch_bounds__(GRP_BLOCK) void k_grp_coarse(
    KeySrc ks, Coarse cm, Lists ls, long nidx, int ipt, uint32_t ncoarse, long nblk, uint32_t ichunk,
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ total, GrpRec* __restrict__ rec,
    uint32_t* __restrict__ base, u32x4* __restrict__ desc, uint32_t* __restrict__ nchunks) {
    extern __shared__ uint32_t cur[];
    __shared__ uint32_t sh[GRP_BLOCK / 64];
    if (long(blockIdx.x) == nblk) {
        grp_plan_block(cm, ls, total, ncoarse, ichunk, base, desc, nchunks, sh);
        return;
    }
    const uint32_t blk = grp_block(nblk);
    // first slot of every range, then of this block's share of it
    for (uint32_t c = threadIdx.x; c < ncoarse; c += GRP_BLOCK) cur[c] = total[c];
    __syncthreads();
    {
        const uint32_t per = (ncoarse + GRP_BLOCK - 1) / GRP_BLOCK;
        const uint32_t c0 = threadIdx.x * per;
        uint32_t n = 0;
        for (uint32_t q = 0; q < per; ++q)
            if (c0 + q < ncoarse) n += cur[c0 + q];
        uint32_t all;
        uint32_t run = block_scan<GRP_BLOCK>(n, sh, &all);
        for (uint32_t q = 0; q < per; ++q)
            if (c0 + q < ncoarse) {
                const uint32_t v = cur[c0 + q];
                cur[c0 + q] = run;
                run += v;
            }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < ncoarse; c += GRP_BLOCK) cur[c] += counts[long(blk) * ncoarse + c];
    __syncthreads();
    const long b0 = long(blk) * ipt * GRP_BLOCK;
    // GRP_UNROLL slots per step: all their loads are issued before any of
    // their records is written
    for (int q0 = 0; q0 < ipt; q0 += GRP_UNROLL) {
        typename KeySrc::Slot sl[GRP_UNROLL];
        bool have[GRP_UNROLL];
#pragma unroll
        for (int u = 0; u < GRP_UNROLL; ++u) {
            const long i = b0 + long(q0 + u) * GRP_BLOCK + threadIdx.x;
            have[u] = ks.fetch(min(i, nidx - 1), sl[u]) && q0 + u < ipt && i < nidx;
        }
#pragma unroll
        for (int u = 0; u < GRP_UNROLL; ++u) {
            if (!have[u]) continue;
            GrpPlace pl;
            ks.place(sl[u], pl);
            const uint32_t d = atomicAdd(&cur[pl.coarse], 1u);
            u32x4* r = reinterpret_cast<u32x4*>(rec + d);
            if constexpr (PACK) {
                const uint32_t cw = pl.ok ? pack_cell(pl.cell) : NO_CELL;
                r[0] = u32x4{pl.key, sl[u].local, __float_as_uint(float(pl.t[0])), __float_as_uint(float(pl.t[1]))};
                r[1] = u32x4{__float_as_uint(float(pl.t[2])), cw, 0u, 0u};
            } else {
                const unsigned long long x0 = __double_as_longlong(sl[u].x[0]);
                const unsigned long long x1 = __double_as_longlong(sl[u].x[1]);
                const unsigned long long x2 = __double_as_longlong(sl[u].x[2]);
                r[0] = u32x4{pl.key, sl[u].local, uint32_t(x0), uint32_t(x0 >> 32)};
                r[1] = u32x4{uint32_t(x1), uint32_t(x1 >> 32), uint32_t(x2), uint32_t(x2 >> 32)};
            }
        }
    }
}

// One binned particle: (PACK) t and the packed cell as 16 bytes, else the
// FP64 position.
template <bool PACK>
__device__ __forceinline__ void grp_put(void* out, uint32_t* perm, uint32_t d, const u32x4& a, const u32x4& b) {
    perm[d] = a.y;
    if constexpr (PACK) {
        static_cast<u32x4*>(out)[d] = u32x4{a.z, a.w, b.x, b.y};
    } else {
        double* x = static_cast<double*>(out) + 3 * long(d);
        x[0] = __longlong_as_double((long long)(uint64_t(a.z) | (uint64_t(a.w) << 32)));
        x[1] = __longlong_as_double((long long)(uint64_t(b.x) | (uint64_t(b.y) << 32)));
        x[2] = __longlong_as_double((long long)(uint64_t(b.z) | (uint64_t(b.w) << 32)));
    }
}

// lh[f], the span's particles of key klo + f, becomes the key's first slot from j0 on;
// the runs' items are written from `slot` on and dealt to the span's `chunks`.
template <typename Lists>
__device__ __forceinline__ void grp_runs(const Lists& ls, u32x4* desc, uint32_t chunks, uint32_t c, uint32_t j0,
                                         uint32_t slot, uint32_t klo, uint32_t nf, uint32_t ichunk,
                                         u32x4* __restrict__ items, uint32_t* lh, uint32_t* sh) {
    // thread t owns the keys [t * per, (t + 1) * per)
    const uint32_t per = (nf + GRP_FINE_BLOCK - 1) / GRP_FINE_BLOCK;
    const uint32_t f0 = threadIdx.x * per;
    const bool emit = ls.wanted(c);
    uint32_t sum = 0, pieces = 0;
    for (uint32_t q = 0; q < per; ++q)
        if (f0 + q < nf) {
            const uint32_t cnt = lh[f0 + q];
            sum += cnt;
            pieces += (cnt + ichunk - 1) / ichunk;
        }
    uint32_t total;
    uint32_t run = block_scan<GRP_FINE_BLOCK>(sum, sh, &total);
    uint32_t at = 0;
    if (emit) {
        at = block_scan<GRP_FINE_BLOCK>(pieces, sh, &total) + slot;
        for (uint32_t i = threadIdx.x; i < chunks; i += GRP_FINE_BLOCK) {
            const uint32_t lo = uint32_t(uint64_t(total) * i / chunks);
            reinterpret_cast<uint32_t*>(desc + i)[2] = uint32_t(uint64_t(total) * (i + 1) / chunks) - lo;
            reinterpret_cast<uint32_t*>(desc + i)[3] = slot + lo;
        }
    }
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t f = f0 + q;
        if (f >= nf) break;
        const uint32_t cnt = lh[f];
        lh[f] = j0 + run;
        if (emit)
            for (uint32_t k = 0; k < cnt; k += ichunk)
                items[at++] = u32x4{ls.origin(c, klo + f), j0 + run + k, min(ichunk, cnt - k), ls.tag(c)};
        run += cnt;
    }
    __syncthreads();
}

// The span of n <= PER * GRP_FINE_BLOCK records (one chunk) from slot j0, keys [klo,
// klo + nf).  All its loads are issued at once.
template <int PER, bool PACK, typename Lists>
__device__ __forceinline__ void grp_sort_chunk(const Lists& ls, const GrpRec* __restrict__ rec, u32x4* desc, uint32_t c,
                                               uint32_t j0, uint32_t n, uint32_t slot, uint32_t klo, uint32_t nf,
                                               uint32_t ichunk, uint32_t* __restrict__ perm, void* __restrict__ out,
                                               u32x4* __restrict__ items, uint32_t* lh, uint32_t* sh) {
    u32x4 a[PER], b[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const u32x4* r = reinterpret_cast<const u32x4*>(rec + j0 + min(q * GRP_FINE_BLOCK + threadIdx.x, n - 1));
        a[q] = load_global16(r);
        b[q] = load_global16(r + 1);
    }
    for (uint32_t f = threadIdx.x; f < nf; f += GRP_FINE_BLOCK) lh[f] = 0;
    __syncthreads();
    // from here on a[q].x is the key from klo on and the record's rank among its equals
    static_assert(GRP_FINE_MAX <= 1u << 13 && PER * GRP_FINE_BLOCK <= 1 << 19, "key and rank in one word");
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * GRP_FINE_BLOCK + threadIdx.x < n) {
            const uint32_t f = a[q].x - klo;
            a[q].x = f | atomicAdd(&lh[f], 1u) << 13;
        }
    __syncthreads();
    grp_runs(ls, desc, PER <= 8 ? 1u : (n + GRP_CHUNK - 1) / GRP_CHUNK, c, j0, slot, klo, nf, ichunk, items, lh, sh);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * GRP_FINE_BLOCK + threadIdx.x < n)
            grp_put<PACK>(out, perm, lh[a[q].x & 0x1fffu] + (a[q].x >> 13), a[q], b[q]);
}

// A longer span: its records are read twice, to count them and to place them.
template <int PER, bool PACK, typename Lists>
__device__ __forceinline__ void grp_sort_span(const Lists& ls, const GrpRec* __restrict__ rec, u32x4* desc, uint32_t c,
                                              uint32_t j0, uint32_t n, uint32_t slot, uint32_t klo, uint32_t nf,
                                              uint32_t ichunk, uint32_t* __restrict__ perm, void* __restrict__ out,
                                              u32x4* __restrict__ items, uint32_t* lh, uint32_t* sh) {
    constexpr uint32_t STEP = PER * GRP_FINE_BLOCK;
    for (uint32_t f = threadIdx.x; f < nf; f += GRP_FINE_BLOCK) lh[f] = 0;
    __syncthreads();
    for (uint32_t s0 = threadIdx.x; s0 < n; s0 += 2 * STEP) {
        uint32_t key[2 * PER];
#pragma unroll
        for (int q = 0; q < 2 * PER; ++q) key[q] = rec[j0 + min(s0 + q * GRP_FINE_BLOCK, n - 1)].key;
#pragma unroll
        for (int q = 0; q < 2 * PER; ++q)
            if (s0 + q * GRP_FINE_BLOCK < n) atomicAdd(&lh[key[q] - klo], 1u);
    }
    __syncthreads();
    grp_runs(ls, desc, (n + GRP_CHUNK - 1) / GRP_CHUNK, c, j0, slot, klo, nf, ichunk, items, lh, sh);
    for (uint32_t s0 = threadIdx.x; s0 < n; s0 += STEP) {
        u32x4 a[PER], b[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const u32x4* r = reinterpret_cast<const u32x4*>(rec + j0 + min(s0 + q * GRP_FINE_BLOCK, n - 1));
            a[q] = load_global16(r);
            b[q] = load_global16(r + 1);
        }
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (s0 + q * GRP_FINE_BLOCK < n)
                grp_put<PACK>(out, perm, atomicAdd(&lh[a[q].x - klo], 1u), a[q], b[q]);
    }
}

template <typename Coarse, typename Lists, bool PACK>
static __global__ __launch_bounds__(GRP_FINE_BLOCK) __attribute__((amdgpu_waves_per_eu(PACK ? 4 : 3))) void k_grp_fine(
    Coarse cm, Lists ls, const GrpRec* __restrict__ rec, u32x4* __restrict__ desc,
    const uint32_t* __restrict__ nchunks, uint32_t ichunk, uint32_t* __restrict__ perm, void* __restrict__ out,
    u32x4* __restrict__ items) {
    extern __shared__ uint32_t lh[];
    __shared__ uint32_t sh[GRP_FINE_BLOCK / 64];
    const uint32_t g = blockIdx.x;
    if (g >= __builtin_amdgcn_readfirstlane(*nchunks)) return;
    const uint32_t c = __builtin_amdgcn_readfirstlane(reinterpret_cast<const uint32_t*>(desc + g)[0]);
    if (c & GRP_FOLLOWS) return;   // (its words 2 and 3 are being written)
    const u32x4 de = desc[g];
    const uint32_t j0 = __builtin_amdgcn_readfirstlane(de.y);
    const uint32_t n = __builtin_amdgcn_readfirstlane(de.z);
    uint32_t klo, khi;
    cm.range(c, klo, khi);
    klo = __builtin_amdgcn_readfirstlane(klo);
    const uint32_t nf = __builtin_amdgcn_readfirstlane(khi) - klo;
    auto sort = [&](auto per) {
        grp_sort_chunk<decltype(per)::value, PACK>(ls, rec, desc + g, c, j0, n, de.w, klo, nf, ichunk, perm, out, items,
                                                   lh, sh);
    };
    if (n <= 4 * GRP_FINE_BLOCK) sort(std::integral_constant<int, 4>{});
    else if (n <= 8 * GRP_FINE_BLOCK) sort(std::integral_constant<int, 8>{});
    else if (n <= GRP_SPAN_REG) sort(std::integral_constant<int, int(GRP_SPAN_REG) / GRP_FINE_BLOCK>{});
    else grp_sort_span<8, PACK>(ls, rec, desc + g, c, j0, n, de.w, klo, nf, ichunk, perm, out, items, lh, sh);
}

// Coarse ranges of a single key space: range c = [c << s, min((c + 1) << s, nb)).
struct ShiftCoarse {
    int s;
    uint32_t nb;
    __device__ __forceinline__ void range(uint32_t c, uint32_t& lo, uint32_t& hi) const {
        lo = c << s;
        hi = min((c + 1) << s, nb);
    }
};

// Shift of ShiftCoarse for P particles over nb keys: about `target`
// particles per coarse range when they are spread evenly, within the LDS
// bounds of both levels.
constexpr uint32_t GRP_TARGET = 512;

inline int grp_shift(uint64_t nb, long P, uint64_t target = GRP_TARGET) {
    int s = 0;
    // smallest s with at most max(P / target, 1) ranges, then the bounds
    const uint64_t want = uint64_t(P) / target > 0 ? uint64_t(P) / target : 1;
    while (((nb + (uint64_t(1) << s) - 1) >> s) > want) ++s;
    while (((nb + (uint64_t(1) << s) - 1) >> s) > GRP_COARSE_MAX) ++s;
    // nb <= (GRP_COARSE_MAX - 1) * GRP_FINE_MAX keeps both bounds
    while ((uint32_t(1) << s) > GRP_FINE_MAX) --s;
    return s;
}

// The most particles (of evenly spread ones) that grp_shift gives a shift of at least
// s > 0: one fewer than make s - 1 few enough ranges.
inline int64_t grp_shift_end(uint64_t nb, int s, uint64_t target = GRP_TARGET) {
    return int64_t(((nb + (uint64_t(1) << (s - 1)) - 1) >> (s - 1)) * target) - 1;
}

// Host-side plan of a grouping of `nidx` slots (nvalid of them particles)
// over the keys [0, nbuckets) in `ncoarse` coarse ranges.
struct GrpPlan {
    long nidx = 0;
    uint32_t nvalid = 0;
    uint32_t nbuckets = 0;
    uint32_t ncoarse = 0;   // coarse ranges
    uint32_t fine_max = 0;  // most keys in one coarse range
    int ipt = 1;            // slots per thread of the coarse passes
    long nblk = 0;          // blocks of the coarse passes
    size_t ncounts = 0;     // counts reserved: never fewer for more particles
    uint32_t mmax = 0;      // most chunks of the fine pass
};

inline GrpPlan grp_plan(long nidx, uint32_t nvalid, uint32_t nbuckets, uint32_t ncoarse, uint32_t fine_max) {
    GrpPlan g;
    g.nidx = nidx;
    g.nvalid = nvalid;
    g.nbuckets = nbuckets;
    g.ncoarse = ncoarse > 0 ? ncoarse : 1;
    g.fine_max = fine_max;
    // one block per CU up to 8 slots per thread, then two
    const long units = (nidx + GRP_BLOCK - 1) / GRP_BLOCK;
    long ipt = (units + GRP_NBLK_MAX / 2 - 1) / (GRP_NBLK_MAX / 2);
    if (ipt > 8) ipt = std::max<long>(8, (units + GRP_NBLK_MAX - 1) / GRP_NBLK_MAX);
    g.ipt = int(ipt < 1 ? 1 : ipt);
    g.nblk = (units + g.ipt - 1) / g.ipt;
    if (g.nblk == 0) g.nblk = 1;
    g.ncounts = size_t(g.ncoarse) * size_t(std::min<long>(std::max<long>(units, 1), GRP_NBLK_MAX));
    // sum over ranges of ceil(n_c / GRP_CHUNK) <= nvalid / GRP_CHUNK + ncoarse
    g.mmax = nvalid / GRP_CHUNK + std::min(g.ncoarse, nvalid);
    return g;
}

// log2 of the units per chunk for about `items` items in all (evenly spread particles).
// Eight: where there are many chunks a unit is then mostly a row of four tiles; four
// for order 4 where a chunk has few items, since a unit costs as much as a cheap item
// (10^6 particles, four / eight units: 128^3 uniform, order 4 FP32 78 / 84, BF16 79 /
// 112 us, clustered 97 / 97, 98 / 126; order 6 clustered FP32 140 / 130, FP64 353 / 335,
// its items being worth balancing).  More while fewer than `target` units come out,
// so that every CU gets some, of three items at least: one of fewer is not yet there
// when the one before ends (64^3 order 4, four / sixteen: FP32 61 / 85, BF16 50 / 105).
inline uint32_t item_units_log2(const GrpPlan& g, uint32_t ichunk, uint32_t target, bool cheap) {
    const uint64_t chunks = std::max<uint64_t>(1, std::max(g.nvalid / GRP_CHUNK, std::min(g.ncoarse, g.nvalid)));
    const uint64_t tiles = std::min(g.nbuckets, g.nvalid);
    const uint64_t items = std::max(tiles, g.nvalid / ichunk + tiles / 2);
    uint32_t l = cheap && items < 16 * chunks ? 2 : 3;
    while (l < 6 && (chunks << l) < target && 3 * (chunks << (l + 1)) <= items) ++l;
    return l;
}

// Most work items of a grouping: a run per span and key present, and one more per
// `ichunk` particles.  A range has one span that is not full; the full ones hold
// GRP_SPAN_RUN particles or more per key, or GRP_SPAN_MAX.
inline size_t grp_item_cap(const GrpPlan& g, uint32_t ichunk) {
    const size_t full = size_t(g.nvalid / GRP_SPAN_MAX) * g.fine_max + g.nvalid / GRP_SPAN_RUN;
    const size_t runs = size_t(g.nbuckets) + full;
    return std::min(runs, size_t(g.nvalid)) + size_t(g.nvalid) / ichunk + 1;
}

// Scratch of a grouping, in uint32 words: records (8 words per particle) and
// chunk descriptors (4 each), both 16-byte aligned like the scratch itself,
// counts, totals and first slots of the ranges, the chunk count.
inline size_t grp_scratch_words(const GrpPlan& g) {
    return 8 * size_t(g.nvalid) + 4 * size_t(g.mmax) + g.ncounts + 2 * size_t(g.ncoarse) + 2;
}

// Device buffers of a grouping, carved from its scratch.
struct GrpBuffers {
    GrpRec* rec;
    u32x4* desc;
    uint32_t *counts, *total, *base, *nchunks;
};

inline GrpBuffers grp_buffers(const GrpPlan& g, uint32_t* scratch) {
    GrpBuffers b;
    b.rec = reinterpret_cast<GrpRec*>(scratch);
    b.desc = reinterpret_cast<u32x4*>(scratch + 8 * size_t(g.nvalid));
    b.counts = scratch + 8 * size_t(g.nvalid) + 4 * size_t(g.mmax);
    b.total = b.counts + g.ncounts;
    b.base = b.total + g.ncoarse;
    b.nchunks = b.base + g.ncoarse + 1;
    return b;
}

// The steps of a grouping, enqueued on one stream.  grp_count also clears
// the nctl control words at ctl.
template <typename KeySrc>
inline void grp_count(const KeySrc& ks, const GrpPlan& g, const GrpBuffers& b, uint32_t* ctl, int nctl,
                      hipStream_t st) {
    hipLaunchKernelGGL((k_grp_hist<KeySrc>), dim3(unsigned(g.nblk)), dim3(GRP_BLOCK),
                       size_t(g.ncoarse) * sizeof(uint32_t), st, ks, g.nidx, g.ipt, g.ncoarse, g.nblk, b.counts, ctl,
                       nctl);
}

inline void grp_scan(const GrpPlan& g, const GrpBuffers& b, hipStream_t st) {
    hipLaunchKernelGGL(k_grp_scan, dim3((g.ncoarse + 63) / 64), dim3(1024), 0, st, b.counts, uint32_t(g.nblk),
                       g.ncoarse, b.total);
}

template <bool PACK, typename KeySrc, typename Coarse, typename Lists>
inline void grp_coarse(const KeySrc& ks, const Coarse& cm, const Lists& ls, const GrpPlan& g, const GrpBuffers& b,
                       uint32_t ichunk, hipStream_t st) {
    hipLaunchKernelGGL((k_grp_coarse<KeySrc, Coarse, Lists, PACK>), dim3(unsigned(g.nblk) + 1), dim3(GRP_BLOCK),
                       size_t(g.ncoarse) * sizeof(uint32_t), st, ks, cm, ls, g.nidx, g.ipt, g.ncoarse, g.nblk,
                       ichunk, b.counts, b.total, b.rec, b.base, b.desc, b.nchunks);
}

// perm and out (nvalid slots each) and, where the lists want them, the items.
template <bool PACK, typename KeySrc, typename Coarse, typename Lists>
inline void grp_scatter(const KeySrc& ks, const Coarse& cm, const Lists& ls, const GrpPlan& g, const GrpBuffers& b,
                        uint32_t ichunk, uint32_t* perm, void* out, u32x4* items, hipStream_t st) {
    grp_coarse<PACK>(ks, cm, ls, g, b, ichunk, st);
    hipLaunchKernelGGL((k_grp_fine<Coarse, Lists, PACK>), dim3(g.mmax), dim3(GRP_FINE_BLOCK),
                       size_t(g.fine_max) * sizeof(uint32_t), st, cm, ls, b.rec, b.desc, b.nchunks, ichunk, perm, out,
                       items);
}

// ----------------------------------------------------------------- gather ---

template <typename CT>
struct Acc {
    using type = float;
};
template <>
struct Acc<double> {
    using type = double;
};

template <typename CT, typename AT>
__device__ __forceinline__ AT widen(CT v) {
    if constexpr (sizeof(CT) == 2) return AT(__uint_as_float(uint32_t(v) << 16));
    else return AT(v);
}

// w_j(t) = sum_i M[j][i] t^i and w'_j(t) = sum_i M1[j][i] t^i (Horner), with
// the matrices of a compile-time table (M from the Section 7 general formula
// for the B-spline).
template <int N, typename AT, typename Tab = BSpline<N>>
__device__ __forceinline__ void bspline_weights(AT t, AT* w, AT* wd) {
    constexpr Tab B{};
#pragma unroll
    for (int j = 0; j < N; ++j) {
        AT acc = AT(B.M[j][N - 1]);
#pragma unroll
        for (int i = N - 2; i >= 0; --i) acc = fused(acc, t, AT(B.M[j][i]));
        w[j] = acc;
        AT dacc = AT(B.M1[j][N - 2]);
#pragma unroll
        for (int i = N - 3; i >= 0; --i) dacc = fused(dacc, t, AT(B.M1[j][i]));
        wd[j] = dacc;
    }
}

// The method's weights (Section 2: w = M tbar, w' = M^(1) tbar): the B-spline
// (the paper's method), Lagrange (N = 2: linear) or, for N = 4, cubic Hermite.
// `basis` is the same for every lane of a launch.
template <int N, typename AT>
__device__ __forceinline__ void basis_weights(int basis, AT t, AT* w, AT* wd) {
    if (basis == BSI_BASIS_LAGRANGE) {
        bspline_weights<N, AT, LagrangeM<N>>(t, w, wd);
    } else {
        if constexpr (N == 4) {
            if (basis == BSI_BASIS_HERMITE) {
                bspline_weights<4, AT, HermiteM>(t, w, wd);
                return;
            }
        }
        bspline_weights<N, AT>(t, w, wd);
    }
}

// The work items a tiled gather reads: those of the chunks [*g0, *g1) (g0 null:
// from the first).
struct ItemSource {
    const u32x4* items;
    const u32x4* desc;
    const uint32_t *g0, *g1;
    uint32_t* ctl;       // take counters (ITEM_CTL_WORDS)
    uint32_t ulog;       // 2^ulog units per chunk
};

inline ItemSource item_source(const BinArrays& b) {
    return ItemSource{static_cast<const u32x4*>(b.items), static_cast<const u32x4*>(b.desc), nullptr, b.nchunks, b.ctl,
                      b.units_log2};
}

struct GatherArgs {
    const void* grid;
    const double* pos;
    const uint32_t* perm;    // binned order, or nullptr
    const void* binned;      // the particles in binned order (RawParticle), or nullptr
    void* u;
    void* grad;
    unsigned long long* nonfinite;
    long P;
    int n0, n1, n2;
    int P1;      // padded extent of axis 1
    int pitch2;  // elements between consecutive (p0, p1) rows of the grid
    double ih0, ih1, ih2;
    int xcd_remap;
    int basis;   // bsi_basis of the field
    int cs;      // stored grid entries per cell along an axis: 1, or 2 for Hermite (direct gather only)
    ItemSource src;      // work items (tiled kernel)
};

__device__ __forceinline__ long logical_block(int remap) {
    const long b = blockIdx.x;
    if (!remap) return b;
    // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD one
    // contiguous range of logical blocks (a compact region of binned particles).
    const long B = gridDim.x;
    const long q = B / 8, r = B % 8;
    const long x = b % 8, i = b / 8;
    return x * q + (x < r ? x : r) + i;
}

template <typename AT, int C, bool GRAD>
__device__ __forceinline__ void write_nan(const GatherArgs& a, long p) {
    const AT nan = AT(__builtin_nan(""));
    AT* u = static_cast<AT*>(a.u) + p * C;
#pragma unroll
    for (int c = 0; c < C; ++c) u[c] = nan;
    if constexpr (GRAD) {
        AT* g = static_cast<AT*>(a.grad) + p * C * 3;
#pragma unroll
        for (int c = 0; c < 3 * C; ++c) g[c] = nan;
    }
}

// A particle of the binned order as it is loaded: for FP32 weights its offsets
// in the cell (FP64 arithmetic, rounded once) and the packed cell, 16 bytes; for
// FP64 its position.
template <typename AT>
struct RawParticle {
    static constexpr bool PACK = true;
    u32x4 r;
    __device__ __forceinline__ void load(const void* binned, long j) {
        r = load_global16(static_cast<const u32x4*>(binned) + j);
    }
    // the compiler waits here for the loads of this particle and its index
    __device__ __forceinline__ void settle(uint32_t& p) { asm volatile("" : "+v"(r), "+v"(p)); }
};
template <>
struct RawParticle<double> {
    static constexpr bool PACK = false;
    double x[3];
    __device__ __forceinline__ void load(const void* binned, long j) {
        const double* p = static_cast<const double*>(binned) + 3 * j;
        x[0] = p[0];
        x[1] = p[1];
        x[2] = p[2];
    }
    __device__ __forceinline__ void settle(uint32_t& p) {
        asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(p));
    }
};

// Cell and offset of the particle at x (Section 5 stencil); false without one.
template <typename AT>
__device__ __forceinline__ bool locate(const double* x, const int* n, const double* ih, int* cell, AT* t) {
    bool ok = true;
    double td[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) ok = cell_of(x[d], ih[d], n[d], cell[d], td[d]) && ok;
#pragma unroll
    for (int d = 0; d < 3; ++d) t[d] = AT(td[d]);
    return ok;
}
__device__ __forceinline__ bool locate(const RawParticle<float>& p, const int*, const double*, int* cell, float* t) {
    cell[0] = int(p.r.w >> 20);
    cell[1] = int((p.r.w >> 10) & 1023u);
    cell[2] = int(p.r.w & 1023u);
    t[0] = __uint_as_float(p.r.x);
    t[1] = __uint_as_float(p.r.y);
    t[2] = __uint_as_float(p.r.z);
    return p.r.w != NO_CELL;
}
__device__ __forceinline__ bool locate(const RawParticle<double>& p, const int* n, const double* ih, int* cell,
                                       double* t) {
    return locate<double>(p.x, n, ih, cell, t);
}

// Weights of a particle with offsets t (Section 2).
template <int N, typename AT>
__device__ __forceinline__ void particle_weights(const GatherArgs& a, const AT* t, AT (*w)[N], AT (*wd)[N]) {
    const double ih[3] = {a.ih0, a.ih1, a.ih2};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        basis_weights<N, AT>(a.basis, t[d], w[d], wd[d]);
        const AT s = AT(ih[d]);
#pragma unroll
        for (int k = 0; k < N; ++k) wd[d][k] *= s;
    }
}

// Tensor contraction of the N^3 (x C) local coefficients with the weights.
// Order follows the Table 1 idea (reduce the tensor order as early as
// possible): each contiguous row of N points along axis 2 is reduced with w2
// and w2' first, then axis 1 with w1 / w1', then axis 0.  The axis-0 sum is
// split into two fixed halves (ia < N/2 and ia >= N/2) that are added at the
// end, so that one particle can also be shared by two lanes; every gather
// variant uses exactly this arithmetic, so their results are bitwise equal.
// `row(ia, ib)` returns a pointer to the N*C coefficients of row (ia, ib).
template <typename AT, int C>
struct Partial {
    AT u[C], g0[C], g1[C], g2[C];
};

// Raw values of one stencil row (N points x C components along axis 2) held
// in registers between their LDS read and their use.  BF16 rows in LDS start
// on 2-byte boundaries, and unaligned wide LDS reads are slow: they are read
// as aligned dwords from the dword boundary at or below the row start and
// realigned by a funnel shift per pair of values when used.  The N*C/2 + 1
// dwords end at most 4 bytes past the row's values, inside the row's padding
// to whole 16-byte chunks for every tile geometry of the tiled gathers.
// PS is the LDS pitch of one grid point in elements: C for densely packed
// rows; 4 for FP32 three-component points held in 16-byte slots, read with one
// 16-byte LDS read each (element e = point e / 3, component e % 3).
template <int N, typename CT, int C, int PS = C>
struct LdsRow {
    static_assert(PS == C, "padded points: FP32, three components");
    CT raw[N * C];
    __device__ __forceinline__ void load(const CT* r) {
#pragma unroll
        for (int e = 0; e < N * C; ++e) raw[e] = r[e];
    }
    __device__ __forceinline__ CT get(int e) const { return raw[e]; }
};

template <int N>
struct LdsRow<N, float, 3, 4> {
    f32x4 pt[N];
    __device__ __forceinline__ void load(const float* r) {
#pragma unroll
        for (int k = 0; k < N; ++k) pt[k] = *reinterpret_cast<const f32x4*>(r + 4 * k);
    }
    __device__ __forceinline__ float get(int e) const { return pt[e / 3][e % 3]; }
};

template <int N, int C>
struct LdsRow<N, uint16_t, C, C> {
    static_assert((N * C) % 2 == 0, "BF16 rows are read as pairs");
    static constexpr int ND = N * C / 2 + 1;
    uint32_t dw[ND];
    uint32_t mis;  // the row's misalignment in bits: 0 or 16
    __device__ __forceinline__ void load(const uint16_t* r) {
        const uint32_t m = uint32_t(reinterpret_cast<uintptr_t>(r)) & 2u;
        const uint32_t* d = reinterpret_cast<const uint32_t*>(r - (m >> 1));
        mis = m * 8u;
#pragma unroll
        for (int k = 0; k < ND; ++k) dw[k] = d[k];
    }
    __device__ __forceinline__ uint16_t get(int e) const {
        const uint32_t v = __builtin_amdgcn_alignbit(dw[e / 2 + 1], dw[e / 2], mis);
        return uint16_t((e & 1) ? (v >> 16) : (v & 0xffffu));
    }
};

// The axis-1/axis-2 sums of one axis-0 plane: v = sum_ib w1[ib] (sum_e w2[e] row[e]),
// with v1 (w1') and v2 (w2') for the gradient.
template <typename AT, int C>
struct PlaneSum {
    AT v[C], v1[C], v2[C];
};

// A row in global memory read value by value (the compiler merges FP32 and FP64
// values into wide loads; BF16 ones stay 2-byte loads).
template <int N, typename CT, int C>
struct PlainRow {
    CT raw[N * C];
    __device__ __forceinline__ void load(const CT* r) {
#pragma unroll
        for (int e = 0; e < N * C; ++e) raw[e] = r[e];
    }
    __device__ __forceinline__ CT get(int e) const { return raw[e]; }
};

// One plane from rows row(ib), ib < N, in global memory, each read as a Row: the
// loads are left to the compiler, which issues them all before the first sum.
template <int N, typename CT, typename AT, int C, bool GRAD, typename Row, typename PlaneRowFn>
__device__ __forceinline__ void plane_sum(const AT (*w)[N], const AT (*wd)[N], PlaneRowFn row, PlaneSum<AT, C>& V) {
#pragma unroll
    for (int c = 0; c < C; ++c) V.v[c] = V.v1[c] = V.v2[c] = AT(0);
#pragma unroll
    for (int ib = 0; ib < N; ++ib) {
        Row cur;
        cur.load(row(ib));
        AT tr[C], trd[C];
#pragma unroll
        for (int c = 0; c < C; ++c) tr[c] = trd[c] = AT(0);
#pragma unroll
        for (int e = 0; e < N; ++e) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const AT val = widen<CT, AT>(cur.get(e * C + c));
                tr[c] += w[2][e] * val;
                if constexpr (GRAD) trd[c] += wd[2][e] * val;
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            V.v[c] += w[1][ib] * tr[c];
            if constexpr (GRAD) {
                V.v1[c] += wd[1][ib] * tr[c];
                V.v2[c] += w[1][ib] * trd[c];
            }
        }
    }
}

// PlaneSum of NP consecutive planes from LDS rows row(k, ib), the rows
// software-pipelined as in contract_planes (the same arithmetic, row by row).
template <int N, typename CT, typename AT, int C, bool GRAD, int NP, int PS, typename RowFn>
__device__ __forceinline__ void plane_sums(const AT (*w)[N], const AT (*wd)[N], RowFn row, PlaneSum<AT, C>* V) {
    LdsRow<N, CT, C, PS> buf[2];
    buf[0].load(row(0, 0));
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        AT v[C], v1[C], v2[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = v1[c] = v2[c] = AT(0);
#pragma unroll
        for (int ib = 0; ib < N; ++ib) {
            const int r = k * N + ib;
            if (r + 1 < NP * N) buf[(r + 1) & 1].load(row((r + 1) / N, (r + 1) % N));
            const LdsRow<N, CT, C, PS>& cur = buf[r & 1];
            AT tr[C], trd[C];
#pragma unroll
            for (int c = 0; c < C; ++c) tr[c] = trd[c] = AT(0);
#pragma unroll
            for (int e = 0; e < N; ++e) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const AT val = widen<CT, AT>(cur.get(e * C + c));
                    tr[c] += w[2][e] * val;
                    if constexpr (GRAD) trd[c] += wd[2][e] * val;
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                v[c] += w[1][ib] * tr[c];
                if constexpr (GRAD) {
                    v1[c] += wd[1][ib] * tr[c];
                    v2[c] += w[1][ib] * trd[c];
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if constexpr (GRAD) asm volatile("" : "+v"(v[c]), "+v"(v1[c]), "+v"(v2[c]));
                else asm volatile("" : "+v"(v[c]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            V[k].v[c] = v[c];
            V[k].v1[c] = v1[c];
            V[k].v2[c] = v2[c];
        }
    }
}

// out += plane k's terms (the accumulation step of contract_planes).
template <typename AT, int C, bool GRAD>
__device__ __forceinline__ void chain_add(Partial<AT, C>& out, AT w0k, AT wd0k, const PlaneSum<AT, C>& V) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
        out.u[c] += w0k * V.v[c];
        if constexpr (GRAD) {
            out.g0[c] += wd0k * V.v[c];
            out.g1[c] += w0k * V.v1[c];
            out.g2[c] += w0k * V.v2[c];
        }
    }
}

template <typename AT, int C, bool GRAD>
__device__ __forceinline__ PlaneSum<AT, C> shfl_planesum(const PlaneSum<AT, C>& V, int src) {
    PlaneSum<AT, C> r;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        r.v[c] = __shfl(V.v[c], src, 64);
        if constexpr (GRAD) {
            r.v1[c] = __shfl(V.v1[c], src, 64);
            r.v2[c] = __shfl(V.v2[c], src, 64);
        }
    }
    return r;
}

template <typename AT, int C, bool GRAD>
__device__ __forceinline__ Partial<AT, C> shfl_partial(const Partial<AT, C>& P, int src) {
    Partial<AT, C> r;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        r.u[c] = __shfl(P.u[c], src, 64);
        if constexpr (GRAD) {
            r.g0[c] = __shfl(P.g0[c], src, 64);
            r.g1[c] = __shfl(P.g1[c], src, 64);
            r.g2[c] = __shfl(P.g2[c], src, 64);
        }
    }
    return r;
}

// NIA consecutive axis-0 planes: w0[k], wd0[k] are the axis-0 weights of
// plane k and row(k, ib) its rows; accumulation order is k = 0..NIA-1.
// FENCE (LDS-resident rows): the NIA*N rows are software-pipelined -- the
// LDS reads of row r+1 are issued before the arithmetic of row r, and a
// scheduling fence after each row keeps at most two rows in registers -- so
// that the LDS latency of one row hides behind the FMAs of the previous one.
// Otherwise (rows in global memory) everything is unrolled and left to the
// compiler.  The arithmetic, and its order, is the same in both forms.
template <int N, typename CT, typename AT, int C, bool GRAD, int NIA, bool FENCE = false, int PS = C,
          typename RowFn>
__device__ __forceinline__ void contract_planes(const AT* w0, const AT* wd0, const AT (*w)[N],
                                                const AT (*wd)[N], RowFn row, Partial<AT, C>& out) {
    static_assert(FENCE || PS == C, "rows in global memory are densely packed");
#pragma unroll
    for (int c = 0; c < C; ++c) out.u[c] = out.g0[c] = out.g1[c] = out.g2[c] = AT(0);
    if constexpr (FENCE) {
        LdsRow<N, CT, C, PS> buf[2];
        buf[0].load(row(0, 0));
#pragma unroll
        for (int k = 0; k < NIA; ++k) {
            AT v[C], v1[C], v2[C];
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = v1[c] = v2[c] = AT(0);
#pragma unroll
            for (int ib = 0; ib < N; ++ib) {
                const int r = k * N + ib;
                if (r + 1 < NIA * N) buf[(r + 1) & 1].load(row((r + 1) / N, (r + 1) % N));
                const LdsRow<N, CT, C, PS>& cur = buf[r & 1];
                AT tr[C], trd[C];
#pragma unroll
                for (int c = 0; c < C; ++c) tr[c] = trd[c] = AT(0);
#pragma unroll
                for (int e = 0; e < N; ++e) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const AT val = widen<CT, AT>(cur.get(e * C + c));
                        tr[c] += w[2][e] * val;
                        if constexpr (GRAD) trd[c] += wd[2][e] * val;
                    }
                }
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    v[c] += w[1][ib] * tr[c];
                    if constexpr (GRAD) {
                        v1[c] += wd[1][ib] * tr[c];
                        v2[c] += w[1][ib] * trd[c];
                    }
                }
                // the row's arithmetic is pinned above the fence (the
                // accumulators pass through an empty side-effecting asm);
                // otherwise it may sink below later rows' reads
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (GRAD) asm volatile("" : "+v"(v[c]), "+v"(v1[c]), "+v"(v2[c]));
                    else asm volatile("" : "+v"(v[c]));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                out.u[c] += w0[k] * v[c];
                if constexpr (GRAD) {
                    out.g0[c] += wd0[k] * v[c];
                    out.g1[c] += w0[k] * v1[c];
                    out.g2[c] += w0[k] * v2[c];
                }
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < NIA; ++k) {
            PlaneSum<AT, C> V;
            plane_sum<N, CT, AT, C, GRAD, PlainRow<N, CT, C>>(w, wd, [&](int ib) { return row(k, ib); }, V);
            chain_add<AT, C, GRAD>(out, w0[k], wd0[k], V);
        }
    }
}

template <typename AT, int C, bool GRAD>
__device__ __forceinline__ void store_sum(const GatherArgs& a, long p, const Partial<AT, C>& lo,
                                          const Partial<AT, C>& hi) {
    AT* u = static_cast<AT*>(a.u) + p * C;
#pragma unroll
    for (int c = 0; c < C; ++c) u[c] = lo.u[c] + hi.u[c];
    if constexpr (GRAD) {
        AT* g = static_cast<AT*>(a.grad) + p * C * 3;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            g[3 * c + 0] = lo.g0[c] + hi.g0[c];
            g[3 * c + 1] = lo.g1[c] + hi.g1[c];
            g[3 * c + 2] = lo.g2[c] + hi.g2[c];
        }
    }
}

// FP32 three-component blocks hold one grid point per 16-byte LDS slot (the
// fourth float is spare): a stencil row is then N aligned 16-byte LDS reads
// wherever it starts, where densely packed 12-byte points need 4-byte reads.
template <typename CT, int C>
constexpr bool padded_points() {
    return sizeof(CT) == 4 && C == 3;
}

// LDS copy of the (T+N-1)^3 block of grid points that the particles of a tile of T^3
// cells read: rows along axis 2, either packed densely and padded to whole
// 16-byte chunks (PAD false), or one 16-byte slot per point (PAD true).
template <int N, typename CT, int C, int T, bool PAD = padded_points<CT, C>()>
struct TileGeom {
    static_assert(!PAD || padded_points<CT, C>(), "padded points: FP32, three components");
    static constexpr bool PADDED = PAD;
    static constexpr int R0 = T + N - 1;
    static constexpr int R1 = T + N - 1;
    static constexpr int R2 = T + N - 1;
    static constexpr int VEC = 16 / int(sizeof(CT));                // elements per 16-byte slot
    static constexpr int PS = PAD ? VEC : C;                        // LDS pitch of a point (elements)
    static constexpr int CH = PAD ? R2 : (R2 * C + VEC - 1) / VEC;  // 16-byte slots per row
    static constexpr int LROW = CH * VEC;                           // LDS row pitch (elements)
    static constexpr int PLANE = R1 * CH;                           // 16-byte slots per axis-0 plane
    static constexpr int SLOTS = R0 * PLANE;
    static constexpr int BYTES = SLOTS * 16;
    // packed rows are copied in 16-byte chunks from the block origin, which
    // must then start on a 16-byte boundary inside a grid row; padded points
    // are copied one point (4-byte aligned) per slot
    static constexpr bool ALIGNED = PAD || (T * C * int(sizeof(CT))) % 16 == 0;
};

// v of the lane that the DPP quad permutation CTRL names (lanes of one group of
// four): a vector instruction, where a shuffle goes through the LDS pipe that
// the stencil reads already fill.
template <int CTRL, typename AT>
__device__ __forceinline__ AT quad_lane(AT v) {
    if constexpr (sizeof(AT) == 8) {
        const unsigned long long b = __double_as_longlong(v);
        const uint32_t lo = __builtin_amdgcn_mov_dpp(int(uint32_t(b)), CTRL, 0xf, 0xf, true);
        const uint32_t hi = __builtin_amdgcn_mov_dpp(int(uint32_t(b >> 32)), CTRL, 0xf, 0xf, true);
        return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
    } else {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
    }
}
constexpr int QUAD_XOR1 = 0xb1;  // lanes 1 0 3 2
constexpr int QUAD_XOR2 = 0x4e;  // lanes 2 3 0 1

// Steps of 64 slots that copy one plane of a block.
template <typename G>
constexpr int plane_steps() {
    return (G::PLANE + 63) / 64;
}

// Byte offsets, from DMA_BIAS before a plane's origin in the grid, of the 16 bytes
// that this lane copies to slot k * 64 + lane of the plane, less the k * 1024 that
// the copy adds to both of its addresses: for a packed block the row's next
// 16-byte chunk, for padded points the 16 bytes from the point's first element
// (the point and the first element of the next one).
constexpr uint32_t DMA_BIAS = 8192;
template <typename CT, int C, typename G>
__device__ __forceinline__ void plane_offsets(int pitch2, uint32_t* off) {
#pragma unroll
    for (int k = 0; k < plane_steps<G>(); ++k) {
        const uint32_t sl = k * 64 + (threadIdx.x & 63u);
        off[k] = (sl / G::CH * uint32_t(pitch2) + sl % G::CH * (G::PADDED ? C : G::VEC)) * uint32_t(sizeof(CT)) +
                 DMA_BIAS - k % 4 * 1024u;
    }
}

// The block in LDS: its R0 axis-0 planes stand in a ring, plane i of the tile at
// place (s + i) mod R0, so that the block slides to the next tile along axis 0 by
// replacing only the planes that it does not share.  All members are uniform.
template <typename G, int T>
struct BlockRing {
    uint32_t held = NO_CELL;   // packed first cell of the tile whose block the LDS holds
    int s = 0;
    __device__ __forceinline__ static int wrap(int v) { return v < G::R0 ? v : v - G::R0; }
    // Moves on to the tile at `origin`; the first of its planes that has to be
    // loaded (R0: none).
    __device__ __forceinline__ int advance(uint32_t origin) {
        if (origin == held) return G::R0;
        const bool slide = held != NO_CELL && origin == held + (uint32_t(T) << 20);
        s = slide ? wrap(s + T) : 0;
        held = origin;
        return slide ? G::R0 - T : 0;
    }
};

// Copies 64 consecutive 16-byte slots, global -> LDS, by the DMA path of the load
// unit: from base + off (per lane) + 1024 k to LDS address lds + 1024 k + 16 lane,
// for k < K (at most four).  Written as instructions: for the compiler's builtin
// every later LDS read, of other arrays too, would wait for the copies, and each
// would set the LDS address anew.  They write no register; wait_loads() waits for
// them.  (s_nop: an address that a vector instruction has just written takes five
// wait states.)
template <int K>
__device__ __forceinline__ void copy_slots(const char* base, const uint32_t* off, uint32_t lds) {
    static_assert(K >= 1 && K <= 4, "one to four steps");
    if constexpr (K == 1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(lds), "v"(off[0]), "s"(base) : "memory", "m0");
    else if constexpr (K == 2)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %3\n\t"
                     "global_load_lds_dwordx4 %2, %3 offset:1024"
                     :: "s"(lds), "v"(off[0]), "v"(off[1]), "s"(base) : "memory", "m0");
    else if constexpr (K == 3)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %4\n\t"
                     "global_load_lds_dwordx4 %2, %4 offset:1024\n\tglobal_load_lds_dwordx4 %3, %4 offset:2048"
                     :: "s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2]), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %5\n\t"
                     "global_load_lds_dwordx4 %2, %5 offset:1024\n\tglobal_load_lds_dwordx4 %3, %5 offset:2048\n\t"
                     "global_load_lds_dwordx4 %4, %5 offset:3072"
                     :: "s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory", "m0");
}
// The same for the step k = K alone (in the lanes that are active).
template <int K>
__device__ __forceinline__ void copy_slots_last(const char* base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                 :: "s"(lds), "v"(off), "s"(base), "n"(K * 1024) : "memory", "m0");
}
// Every load of this wavefront has come in (stores have gone out).
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// p, known to be the same in every lane, in scalar registers.
__device__ __forceinline__ const char* uniform(const char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
    return reinterpret_cast<const char*>((uint64_t(hi) << 32) | lo);
}

// Requests the LDS copy of planes [i0, R0) of the block with cell origin (o0, o1,
// o2) in the ghost-padded grid, the wavefronts taking planes in turn.  Planes
// outside the padded grid (partial blocks only; never read by a particle) are
// left out, rows outside it load the plane's origin instead; reads past a row's
// end land in the next row, its pitch padding or the allocation's slack.
template <int N, typename CT, int C, typename G, int T, int B>
__device__ __forceinline__ void block_dma(const void* grid, int n0, int n1, int P1, int pitch2, int o0, int o1,
                                          int o2, const BlockRing<G, T>& ring, int i0, const uint32_t* off,
                                          u32x4* lds) {
    constexpr int Q = plane_steps<G>();
    static_assert(Q <= 8, "a plane is copied in at most two groups of four steps");
    const int lane = threadIdx.x & 63;
    const long plane_bytes = long(P1) * pitch2 * long(sizeof(CT));
    const char* g = static_cast<const char*>(grid) - DMA_BIAS +
                    ((long(o0) * P1 + o1) * pitch2 + long(o2) * C) * long(sizeof(CT));
    const int last = min(n0 + N - 1 - o0, G::R0);
    const int lim1 = n1 + N - 1 - o1;
    const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) u32x4*)lds));
    uint32_t e[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) e[k] = off[k];
    if (lim1 < G::R1) {
#pragma unroll
        for (int k = 0; k < Q; ++k) e[k] = (k * 64 + lane) / G::CH < lim1 ? e[k] : DMA_BIAS - k % 4 * 1024u;
    }
    for (int i = i0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); i < last; i += B / 64) {
        const char* gi = uniform(g + i * plane_bytes);
        const uint32_t dst =
            __builtin_amdgcn_readfirstlane(lds0 + uint32_t(BlockRing<G, T>::wrap(ring.s + i) * G::PLANE * 16));
        constexpr int FULL = G::PLANE / 64;   // steps without masked lanes
        if constexpr (FULL >= 4) copy_slots<4>(gi, e, dst);
        if constexpr (FULL % 4 != 0) copy_slots<FULL % 4>(gi, e + FULL / 4 * 4, dst + FULL / 4 * 4096u);
        if constexpr (Q > FULL)
            if (FULL * 64 + lane < G::PLANE) copy_slots_last<FULL % 4>(gi, e[FULL], dst + FULL / 4 * 4096u);
    }
}

// The aligned dword reads of a BF16 row (LdsRow) stay inside the row's
// LDS pitch for every stencil start dc = 0 .. T2-1 of a T2-cell box.
template <int N, int C, int T2, int LROW>
constexpr bool bf16_rows_fit() {
    for (int dc = 0; dc < T2; ++dc) {
        const int start = 2 * dc * C;
        if (start - start % 4 + 4 * (N * C / 2 + 1) > 2 * LROW) return false;
    }
    return true;
}

// Lanes per particle for `count` particles on W wavefronts: as many as still
// hold all of them in one round (order 6: 6, 3 or 2 lanes of 1, 2 or 3 axis-0
// planes; order 4: 4 or 2; order 2: 2), else one.  A sparse tile's wavefronts
// then finish sooner and read LDS banks that differ between the lanes of a
// particle (planes are an odd number of 16-byte slots apart).
template <int N, int W, bool SIX>
__device__ __forceinline__ int particle_lanes(uint32_t count) {
    if constexpr (N == 6) {
        if (SIX && count <= uint32_t(W * 10)) return 6;
        if (count <= uint32_t(W * 21)) return 3;
    } else if constexpr (N == 4) {
        if (count <= uint32_t(W * 16)) return 4;
    }
    return count <= uint32_t(W * 32) ? 2 : 1;
}

// Particle of this lane among those of one round (j), and its part of the
// particle's axis-0 planes.
struct LaneRole {
    uint32_t j;
    int part;
    bool ok;   // false: a spare lane (64 is no multiple of the lanes per particle)
};
__device__ __forceinline__ LaneRole lane_role(int lanes) {
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    LaneRole r;
    if (lanes == 1) {
        r.j = threadIdx.x;
        r.part = 0;
        r.ok = true;
    } else if (lanes == 2) {
        r.j = threadIdx.x >> 1;
        r.part = lane & 1;
        r.ok = true;
    } else if (lanes == 4) {
        r.j = threadIdx.x >> 2;
        r.part = lane & 3;
        r.ok = true;
    } else if (lanes == 3) {
        r.j = wid * 21 + lane / 3;
        r.part = int(lane % 3);
        r.ok = lane < 63;
    } else {
        r.j = wid * 10 + lane / 6;
        r.part = int(lane % 6);
        r.ok = lane < 60;
    }
    return r;
}

// One particle on SL > 2 neighbouring lanes, N / SL axis-0 planes each: the
// lanes holding planes 0 and N / 2 fetch the other planes of their half from
// the lanes next to them and add them up in the order of contract_planes; the
// sum of the upper half goes to part 0, which stores.
template <int N, typename AT, int C, bool GRAD, int SL>
__device__ __forceinline__ void split_sum(const GatherArgs& a, long p, bool store, int part, const AT (*w)[N],
                                          const AT (*wd)[N], const PlaneSum<AT, C>* V) {
    constexpr int PPL = N / SL, H = N / 2;
    const int lane = threadIdx.x & 63;
    const bool upper = part * PPL >= H;
    AT w0[H], wd0[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        w0[k] = upper ? w[0][H + k] : w[0][k];
        wd0[k] = upper ? wd[0][H + k] : wd[0][k];
    }
    Partial<AT, C> sum;
#pragma unroll
    for (int c = 0; c < C; ++c) sum.u[c] = sum.g0[c] = sum.g1[c] = sum.g2[c] = AT(0);
    if constexpr (SL == 3) {
        // planes 0 1 | 2 3 | 4 5: part 0 takes 2 from part 1, part 2 takes 3
        const PlaneSum<AT, C> X = shfl_planesum<AT, C, GRAD>(V[0], (lane + 1) & 63);
        const PlaneSum<AT, C> Y = shfl_planesum<AT, C, GRAD>(V[1], (lane + 63) & 63);
        auto pick = [&](const PlaneSum<AT, C>& lo, const PlaneSum<AT, C>& hi) {
            PlaneSum<AT, C> r;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                r.v[c] = upper ? hi.v[c] : lo.v[c];
                if constexpr (GRAD) {
                    r.v1[c] = upper ? hi.v1[c] : lo.v1[c];
                    r.v2[c] = upper ? hi.v2[c] : lo.v2[c];
                }
            }
            return r;
        };
        chain_add<AT, C, GRAD>(sum, w0[0], wd0[0], pick(V[0], Y));
        chain_add<AT, C, GRAD>(sum, w0[1], wd0[1], pick(V[1], V[0]));
        chain_add<AT, C, GRAD>(sum, w0[2], wd0[2], pick(X, V[1]));
        const Partial<AT, C> up = shfl_partial<AT, C, GRAD>(sum, (lane + 2) & 63);
        if (store) store_sum<AT, C, GRAD>(a, p, sum, up);
    } else if constexpr (SL == 6) {
        const PlaneSum<AT, C> X = shfl_planesum<AT, C, GRAD>(V[0], (lane + 1) & 63);
        const PlaneSum<AT, C> Y = shfl_planesum<AT, C, GRAD>(V[0], (lane + 2) & 63);
        chain_add<AT, C, GRAD>(sum, w0[0], wd0[0], V[0]);
        chain_add<AT, C, GRAD>(sum, w0[1], wd0[1], X);
        chain_add<AT, C, GRAD>(sum, w0[2], wd0[2], Y);
        const Partial<AT, C> up = shfl_partial<AT, C, GRAD>(sum, (lane + 3) & 63);
        if (store) store_sum<AT, C, GRAD>(a, p, sum, up);
    } else {
        static_assert(SL == 4 && N == 4, "lanes per particle: 3, 4 or 6");
        PlaneSum<AT, C> X;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            X.v[c] = quad_lane<QUAD_XOR1>(V[0].v[c]);
            if constexpr (GRAD) {
                X.v1[c] = quad_lane<QUAD_XOR1>(V[0].v1[c]);
                X.v2[c] = quad_lane<QUAD_XOR1>(V[0].v2[c]);
            }
        }
        chain_add<AT, C, GRAD>(sum, w0[0], wd0[0], V[0]);
        chain_add<AT, C, GRAD>(sum, w0[1], wd0[1], X);
        Partial<AT, C> up;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            up.u[c] = quad_lane<QUAD_XOR2>(sum.u[c]);
            if constexpr (GRAD) {
                up.g0[c] = quad_lane<QUAD_XOR2>(sum.g0[c]);
                up.g1[c] = quad_lane<QUAD_XOR2>(sum.g1[c]);
                up.g2[c] = quad_lane<QUAD_XOR2>(sum.g2[c]);
            }
        }
        if (store) store_sum<AT, C, GRAD>(a, p, sum, up);
    }
}

// The same from the LDS rows of the planes.
template <int N, typename CT, typename AT, int C, bool GRAD, int SL, int PS, typename RowFn>
__device__ __forceinline__ void split_eval(const GatherArgs& a, long p, bool store, int part, const AT (*w)[N],
                                           const AT (*wd)[N], RowFn rows) {
    constexpr int PPL = N / SL;
    PlaneSum<AT, C> V[PPL];
    plane_sums<N, CT, AT, C, GRAD, PPL, PS>(w, wd, [&](int k, int ib) { return rows(part * PPL + k, ib); }, V);
    split_sum<N, AT, C, GRAD, SL>(a, p, store, part, w, wd, V);
}

// One particle on two lanes, a half of the axis-0 planes each.
template <int N, typename CT, typename AT, int C, bool GRAD, int PS, typename RowFn>
__device__ __forceinline__ void pair_eval(const GatherArgs& a, long p, bool store, int half, const AT (*w)[N],
                                          const AT (*wd)[N], RowFn rows) {
    const int ia0 = half * (N / 2);
    AT w0s[N / 2], wd0s[N / 2];
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        w0s[k] = half ? w[0][N / 2 + k] : w[0][k];
        wd0s[k] = half ? wd[0][N / 2 + k] : wd[0][k];
    }
    Partial<AT, C> mine, other;
    contract_planes<N, CT, AT, C, GRAD, N / 2, true, PS>(
        w0s, wd0s, w, wd, [&](int k, int ib) { return rows(ia0 + k, ib); }, mine);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        other.u[c] = quad_lane<QUAD_XOR1>(mine.u[c]);
        if constexpr (GRAD) {
            other.g0[c] = quad_lane<QUAD_XOR1>(mine.g0[c]);
            other.g1[c] = quad_lane<QUAD_XOR1>(mine.g1[c]);
            other.g2[c] = quad_lane<QUAD_XOR1>(mine.g2[c]);
        }
    }
    if (store) store_sum<AT, C, GRAD>(a, p, mine, other);
}

// Particle of slot j in binned order, or of index j when the particles are not
// binned: its index p, cell and fractional position; false when it has none.
template <typename AT>
__device__ __forceinline__ bool direct_particle(const GatherArgs& a, long j, long& p, int* cell, AT* t) {
    const int n[3] = {a.n0, a.n1, a.n2};
    const double ih[3] = {a.ih0, a.ih1, a.ih2};
    p = j;
    if (a.perm) {
        p = long(a.perm[j]);
        RawParticle<AT> raw;
        raw.load(a.binned, j);
        return locate(raw, n, ih, cell, t);
    }
    const double x[3] = {a.pos[3 * j], a.pos[3 * j + 1], a.pos[3 * j + 2]};
    return locate<AT>(x, n, ih, cell, t);
}

// Row (0, 0) of the particle's stencil in the grid.
template <typename CT, int C>
__device__ __forceinline__ const CT* direct_base(const GatherArgs& a, const int* cell) {
    return static_cast<const CT*>(a.grid) + (long(a.cs * cell[0]) * a.P1 + a.cs * cell[1]) * a.pitch2 +
           long(a.cs * cell[2]) * C;
}

// One particle evaluated straight from the grid in global memory (the caches
// provide the reuse between neighbouring binned particles).
template <int N, typename CT, int C, bool GRAD>
__device__ __forceinline__ void direct_eval(const GatherArgs& a, long j) {
    using AT = typename Acc<CT>::type;
    long p;
    int cell[3];
    AT t[3];
    if (!direct_particle(a, j, p, cell, t)) {
        write_nan<AT, C, GRAD>(a, p);
        atomicAdd(a.nonfinite, 1ull);
        return;
    }
    AT w[3][N], wd[3][N];
    particle_weights<N, AT>(a, t, w, wd);
    const CT* base = direct_base<CT, C>(a, cell);
    const long rowA = long(a.P1) * a.pitch2;
    const long rowB = a.pitch2;
    Partial<AT, C> lo, hi;
    auto row = [&](int ia, int ib) { return base + ia * rowA + ib * rowB; };
    contract_planes<N, CT, AT, C, GRAD, N / 2>(w[0], wd[0], w, wd, row, lo);
    contract_planes<N, CT, AT, C, GRAD, N / 2>(w[0] + N / 2, wd[0] + N / 2, w, wd,
                                               [&](int k, int ib) { return row(N / 2 + k, ib); }, hi);
    store_sum<AT, C, GRAD>(a, p, lo, hi);
}

// Weight polynomials by stencil index, highest power first: row j of a basis holds
// those of w_j, then of w_j' (without its chain factor).
template <int N, typename AT>
struct WeightRows {
    static constexpr int ROW = (2 * N - 1 + 3) / 4 * 4;
    AT row[3][N][ROW];   // B-spline, Lagrange, Hermite (N = 4)
    template <typename Basis>
    constexpr void fill(int b) {
        Basis m{};
        for (int j = 0; j < N; ++j) {
            for (int i = 0; i < N; ++i) row[b][j][N - 1 - i] = AT(m.M[j][i]);
            for (int i = 0; i < N - 1; ++i) row[b][j][2 * N - 2 - i] = AT(m.M1[j][i]);
        }
    }
    constexpr WeightRows() : row{} {
        fill<BSpline<N>>(0);
        fill<LagrangeM<N>>(1);
        if constexpr (N == 4) fill<HermiteM>(2);
    }
};
template <int N, typename AT>
__device__ const WeightRows<N, AT> weight_rows{};

// Weight pairs of axes 1 and 2 of a wavefront's particles (the spare lanes of
// order 6 have a slot too).
template <int N, typename AT>
struct SplitSlots {
    AT pair[(63 + N) / N][2][N][2];
};

// Weights of a particle on N lanes: each lane forms those of stencil index `part`
// along the three axes (the Horner steps of bspline_weights) and reads the others'
// through LDS (a wavefront's LDS instructions go in order; a fence and a wave barrier
// between the pairs' writes and reads cost 7 % at 10^3 .. 1.6 * 10^5 particles); w[0][i],
// i < N / 2, is plane i of the lane's half from the lane on (split_sum).
template <int N, typename AT>
__device__ __forceinline__ void split_weights(const GatherArgs& a, const AT* t, int part, AT (*slot)[N][2],
                                              AT (*w)[N], AT (*wd)[N]) {
    const int lane = threadIdx.x & 63;
    const int b = a.basis == BSI_BASIS_LAGRANGE ? 1 : a.basis == BSI_BASIS_HERMITE ? 2 : 0;
    const AT* c = weight_rows<N, AT>.row[b][part];
    const double ih[3] = {a.ih0, a.ih1, a.ih2};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        AT x = c[0], xd = c[N];
#pragma unroll
        for (int q = 1; q < N; ++q) x = fused(x, t[d], c[q]);
#pragma unroll
        for (int q = 1; q < N - 1; ++q) xd = fused(xd, t[d], c[N + q]);
        xd *= AT(ih[d]);
        if (d == 0) {
            w[0][0] = x;
            wd[0][0] = xd;
        } else {
            slot[d - 1][part][0] = x;
            slot[d - 1][part][1] = xd;
        }
    }
#pragma unroll
    for (int d = 1; d < 3; ++d)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            w[d][j] = slot[d - 1][j][0];
            wd[d][j] = slot[d - 1][j][1];
        }
    if constexpr (N == 4) {
        w[0][1] = quad_lane<QUAD_XOR1>(w[0][0]);
        wd[0][1] = quad_lane<QUAD_XOR1>(wd[0][0]);
    } else {
#pragma unroll
        for (int i = 1; i < N / 2; ++i) {
            w[0][i] = __shfl(w[0][0], (lane + i) & 63, 64);
            wd[0][i] = __shfl(wd[0][0], (lane + i) & 63, 64);
        }
    }
#pragma unroll
    for (int i = N / 2; i < N; ++i) {
        w[0][i] = w[0][i - N / 2];
        wd[0][i] = wd[0][i - N / 2];
    }
}

// The same on N neighbouring lanes (N = 4 or 6), one axis-0 plane each: all of a
// particle's rows are requested at once, where one lane works through N times as
// many, and each weight is formed once.  j0 is the wavefront's first particle;
// every lane of it calls this.  A BF16 row is read as aligned dwords, one 16-byte
// load or three instead of 6 or 18 of two bytes; they end at most four bytes past
// the row, and the grid's allocation goes on further (4 KB).
template <int N, typename CT, int C, bool GRAD>
__device__ __forceinline__ void direct_split_eval(const GatherArgs& a, long j0,
                                                  SplitSlots<N, typename Acc<CT>::type>& slots) {
    using AT = typename Acc<CT>::type;
    const int lane = threadIdx.x & 63;
    const int part = lane % N;
    // spare lanes (N = 6: four) and lanes past the end work on the last particle
    // of the wavefront and store nothing
    const bool mine = lane / N < 64 / N && j0 + lane / N < a.P;
    const long j = min(j0 + min(lane / N, 64 / N - 1), a.P - 1);
    long p;
    int cell[3];
    AT t[3];
    const bool ok = direct_particle(a, j, p, cell, t);
    if (!ok) {
        cell[0] = cell[1] = cell[2] = 0;
        t[0] = t[1] = t[2] = AT(0);
        if (mine && part == 0) {
            write_nan<AT, C, GRAD>(a, p);
            atomicAdd(a.nonfinite, 1ull);
        }
    }
    const CT* plane = direct_base<CT, C>(a, cell) + part * (long(a.P1) * a.pitch2);
    AT w[3][N], wd[3][N];
    split_weights<N, AT>(a, t, part, slots.pair[lane / N], w, wd);
    PlaneSum<AT, C> V;
    plane_sum<N, CT, AT, C, GRAD, LdsRow<N, CT, C>>(w, wd, [&](int ib) { return plane + ib * long(a.pitch2); }, V);
    split_sum<N, AT, C, GRAD, N>(a, p, mine && ok && part == 0, part, w, wd, &V);
}

// NaN outputs for the `count` particles without a cell (the last bucket),
// which are also counted.
template <typename AT, int C, bool GRAD, int B>
__device__ __forceinline__ void nonfinite_eval(const GatherArgs& a, uint32_t count, uint32_t start) {
    for (uint32_t j = threadIdx.x; j < count; j += B) write_nan<AT, C, GRAD>(a, long(a.perm[start + j]));
    if (threadIdx.x == 0) atomicAdd(a.nonfinite, (unsigned long long)count);
}

// ------------------------------------------------------- taking items -------

// A workgroup's place in the work items.  It takes units of its home range in
// order, through the range's counter, then those of the other ranges, and is done
// when every range is exhausted.  Which ranges still have units is read for all
// of them at once (eight ranges tried one after another cost a workgroup without
// work eight round trips: 80 instead of 46 us for the 64 tiles of a 32^3 field).
// Units dealt to the workgroups in turn instead of taken: 2232 instead of 1730
// us for 5 * 10^6 particles at 512^3 (the workgroups do not keep step).
//
// The next unit is fetched while the items of the current one are evaluated, one
// step (counter, descriptor, items) per item, each when the loads of the step
// before have come in anyway; the items themselves stand in the lanes of a
// register.  All other members are the same in every lane, and every thread of
// the workgroup calls every function.
template <int B>
struct ItemStream {
    ItemSource s;
    uint32_t* sh;        // three LDS words (B > 64)
    uint32_t gbeg, nch;  // chunks [gbeg, gbeg + nch)
    uint32_t x;          // current range
    uint32_t xbeg, xend; // its first chunk, and its units
    uint32_t xadd;       // its units that workgroups start on: the counter counts from there
    u32x4 its;           // lane l: item base + l
    uint32_t base, k, m; // items [base + k, base + m) are left of the unit
    int stage;           // of the next unit: 1 counter, 2 descriptor, 3 items requested, 4 here, 5 none left
    uint32_t v;          // stage 1: the counter's value (first lane)
    bool spread;         // workgroup b's home is range b mod ITEM_RANGES (else 0 for all)
    u32x4 q;             // stage 2: the descriptor, 3 and 4: lane l: item nbase + l
    uint32_t nbase, nm;

    // The first item into it; false when there is none at all.
    __device__ __forceinline__ bool begin(const ItemSource& src, uint32_t* lds, bool homes_spread, u32x4& it) {
        s = src;
        sh = lds;
        // the first unit needs no counter: the workgroups of a range start on its first ones
        spread = homes_spread;
        x = spread ? blockIdx.x % ITEM_RANGES : 0u;
        stage = 1;
        gbeg = s.g0 ? __builtin_amdgcn_readfirstlane(*s.g0) : 0u;
        nch = __builtin_amdgcn_readfirstlane(*s.g1) - gbeg;
        enter();
        v = (spread ? blockIdx.x / ITEM_RANGES : blockIdx.x) - xadd;
        k = m = 0;
        return next_wait(it);
    }
    // After a wait for all loads: the compiler needs no further one for these.
    __device__ __forceinline__ void settle() { asm volatile("" : "+v"(v), "+v"(q)); }
    // Before a barrier that follows a wait for all loads ...
    __device__ __forceinline__ void publish() {
        if constexpr (B > 64)
            if (stage == 1 && threadIdx.x == 0) sh[0] = v;
    }
    // ... and after it.
    __device__ __forceinline__ void step() {
        const u32x4* from = s.items;
        uint32_t last = 0;
        int load = 0;
        if (stage == 1) {
            uint32_t unit = __builtin_amdgcn_readfirstlane(B > 64 ? sh[0] : v) + xadd;
            if (unit >= xend && !seek(unit)) {
                stage = 5;
            } else {
                nm = unit & ((1u << s.ulog) - 1u);   // until the descriptor is here
                from = s.desc + xbeg + (unit >> s.ulog);
                load = 1;
                stage = 2;
            }
        } else if (stage == 2) {
            const uint32_t n = __builtin_amdgcn_readfirstlane(q.z), first = __builtin_amdgcn_readfirstlane(q.w);
            const uint32_t lo = (n * nm) >> s.ulog, hi = (n * (nm + 1)) >> s.ulog;
            nbase = first + lo;
            nm = hi - lo;
            if (nm == 0) {
                request();
            } else {
                from += nbase;
                last = nm - 1;
                load = 1;
                stage = 3;
            }
        } else if (stage == 3) {
            stage = 4;
        }
        // One load in one place (the compiler is not to move it into the branches):
        // where branches that load meet, it copies what they loaded, and waits for it
        // (256^3, 10^6: order 6 255 -> 240 us an evaluation, second derivatives 360 ->
        // 344; 512^3, 10^7 clustered, BF16 1955 -> 1895).
        asm volatile("" : "+s"(load));
        if (load) q = load_global16(from + min(threadIdx.x & 63u, last));
    }
    // The next item into it without waiting for any; false: not known yet (or
    // there is none).
    __device__ __forceinline__ bool next(u32x4& it) {
        if (k + 1 < m && k + 1 < 64) {
            ++k;
        } else if (k + 1 >= m && stage == 4) {
            start_unit();
        } else {
            return false;
        }
        it = item();
        return true;
    }
    // The next item into it; false when all ranges are exhausted.
    __device__ __forceinline__ bool next_wait(u32x4& it) {
        if (k + 1 < m) {   // past the 64 items of the register
            base += k + 1;
            m -= k + 1;
            k = 0;
            its = fetch(base, m);
        } else {
            while (stage < 4) {
                __builtin_amdgcn_s_waitcnt(0);
                publish();
                if constexpr (B > 64) __syncthreads();
                step();
                if constexpr (B > 64) __syncthreads();   // sh may be written again
            }
            if (stage == 5) return false;
            start_unit();
        }
        it = item();
        return true;
    }

   private:
    __device__ __forceinline__ u32x4 item() const {
        return u32x4{uint32_t(__builtin_amdgcn_readlane(its.x, k)), uint32_t(__builtin_amdgcn_readlane(its.y, k)),
                     uint32_t(__builtin_amdgcn_readlane(its.z, k)), uint32_t(__builtin_amdgcn_readlane(its.w, k))};
    }
    __device__ __forceinline__ void request() {
        v = threadIdx.x == 0 ? atomicAdd(s.ctl + ITEM_CTL_STRIDE * x, 1u) : 0u;
        stage = 1;
    }
    // Units of range r that workgroups start on.
    __device__ __forceinline__ uint32_t firsts(uint32_t r) const {
        return spread ? (gridDim.x + ITEM_RANGES - 1 - r) / ITEM_RANGES : r == 0 ? gridDim.x : 0u;
    }
    __device__ __forceinline__ u32x4 fetch(uint32_t from, uint32_t n) const {
        return load_global16(s.items + from + min(threadIdx.x & 63u, n - 1));
    }
    __device__ __forceinline__ void start_unit() {
        its = q;
        base = nbase;
        m = nm;
        k = 0;
        request();
    }
    __device__ __forceinline__ uint32_t units(uint32_t r) const {
        return (item_range_begin(r + 1, nch) - item_range_begin(r, nch)) << s.ulog;
    }
    // A unit of another range that still has some; false when none has.
    __device__ __forceinline__ bool seek(uint32_t& unit) {
        if constexpr (B > 64) {
            // the first wavefront looks for all (they must agree)
            if (threadIdx.x < 64) {
                seek_wave(unit);
                sh[1] = x;
                sh[2] = unit;
            }
            __syncthreads();
            x = __builtin_amdgcn_readfirstlane(sh[1]);
            unit = __builtin_amdgcn_readfirstlane(sh[2]);
            __syncthreads();
        } else {
            seek_wave(unit);
        }
        if (x == ITEM_RANGES) return false;
        enter();
        return true;
    }
    __device__ __forceinline__ void enter() {
        xbeg = gbeg + item_range_begin(x, nch);
        xend = units(x);
        xadd = firsts(x);
    }
    // One wavefront; counters only grow, so the loop ends.
    __device__ __forceinline__ void seek_wave(uint32_t& unit) {
        for (;;) {
            const uint32_t l = threadIdx.x % ITEM_RANGES;
            const uint32_t at =
                __hip_atomic_load(s.ctl + ITEM_CTL_STRIDE * l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t some = uint32_t(__ballot(at + firsts(l) < units(l))) & ((1u << ITEM_RANGES) - 1u);
            if (some == 0) {
                x = ITEM_RANGES;
                return;
            }
            const uint32_t turn = (x + 1) % ITEM_RANGES;
            x = (turn + uint32_t(__builtin_ctz((some | (some << ITEM_RANGES)) >> turn))) % ITEM_RANGES;
            // (not by request(): stage must stay the same in every wavefront)
            v = threadIdx.x == 0 ? atomicAdd(s.ctl + ITEM_CTL_STRIDE * x, 1u) : 0u;
            unit = __builtin_amdgcn_readfirstlane(v) + firsts(x);
            if (unit < units(x)) return;
        }
    }
};

// Called once by every workgroup when all ranges are exhausted: the last one
// sets the take counters back, so that another run over the same items needs no
// launch to do it.  The workgroups are counted in groups, and the groups: one counter
// takes about 15 ns a workgroup, which held up the end of every run (32768 items at
// 256^3 on 3072 workgroups, BF16 order 4: 117 us, 109 in groups, 104 when the first
// units need no counter either).
__device__ __forceinline__ void item_take_end(uint32_t* ctl) {
    if (threadIdx.x != 0) return;
    const uint32_t g = blockIdx.x % ITEM_GROUPS;
    const uint32_t groups = min(gridDim.x, uint32_t(ITEM_GROUPS));
    const uint32_t members = (gridDim.x - g + ITEM_GROUPS - 1) / ITEM_GROUPS;
    uint32_t* done = ctl + ITEM_CTL_STRIDE * ITEM_RANGES;
    uint32_t* all = done + ITEM_CTL_STRIDE * ITEM_GROUPS;
    if (atomicAdd(done + ITEM_CTL_STRIDE * g, 1u) + 1 != members) return;
    atomicExch(done + ITEM_CTL_STRIDE * g, 0u);
    if (atomicAdd(all, 1u) + 1 != groups) return;
    for (int x = 0; x < ITEM_RANGES; ++x) atomicExch(ctl + ITEM_CTL_STRIDE * x, 0u);
    atomicExch(all, 0u);
}

// Weight pairs (w, w') of a particle on several lanes, through LDS: every lane
// forms those of its own stencil indices along the three axes and reads the
// others', where forming all of them in every lane took half of a sparse tile's
// vector instructions.  The Horner steps and the coefficients are those of
// bspline_weights, so the weights are the same to the last bit.
template <int N, typename AT, int W>
struct SharedWeights {
    // row j: M[j][N-1 .. 0], then M1[j][N-2 .. 0] (w' without its chain factor)
    static constexpr int ROW = (2 * N - 1 + 3) / 4 * 4;
    AT coef[N][ROW];
    // pairs of axes 1 and 2 of the particles of a round; SPW of them per wavefront
    static constexpr int SPW = N == 6 ? 22 : 16;   // (order 6: the spare lane has its own)
    AT pair[W][SPW][2][N][2];
};

// What a tiled kernel does with one particle: value and gradient.
template <int N_, typename CT_, int C_, bool GRAD, int T_, int W_>
struct ValueGather {
    static constexpr int N = N_, C = C_, T = T_;
    using CT = CT_;
    using AT = typename Acc<CT>::type;
    using G = TileGeom<N, CT, C, T>;
    using Args = GatherArgs;
    static constexpr bool SHARE = sizeof(AT) == 4 && N >= 4;
    struct Empty {};
    using Shared = typename std::conditional<SHARE, SharedWeights<N, AT, W_>, Empty>::type;
    struct Weights {
        AT w[3][N], wd[3][N];
    };
    template <int W>
    __device__ __forceinline__ static int lanes(uint32_t count) {
        return particle_lanes<N, W, SHARE>(count);
    }
    __device__ __forceinline__ static void init(const Args& a, Shared* sh) {
        if constexpr (SHARE) {
            constexpr BSpline<N> S{};
            constexpr LagrangeM<N> L{};
            if (threadIdx.x == 0) {
                const bool lag = a.basis == BSI_BASIS_LAGRANGE;
#pragma unroll
                for (int j = 0; j < N; ++j) {
#pragma unroll
                    for (int i = 0; i < N; ++i) sh->coef[j][N - 1 - i] = lag ? AT(L.M[j][i]) : AT(S.M[j][i]);
#pragma unroll
                    for (int i = 0; i < N - 1; ++i) sh->coef[j][2 * N - 2 - i] = lag ? AT(L.M1[j][i]) : AT(S.M1[j][i]);
                }
            }
            __syncthreads();
        }
    }
    __device__ __forceinline__ static void setup(const Args& a, const RawParticle<AT>& raw, int lanes,
                                                 const LaneRole& role, int* cell, Weights& k, Shared* sh) {
        const int n[3] = {a.n0, a.n1, a.n2};
        const double ih[3] = {a.ih0, a.ih1, a.ih2};
        AT t[3];
        locate(raw, n, ih, cell, t);   // finite by construction of the bucket
        if constexpr (SHARE) {
            if (lanes > 2) {
                if (N == 4 || lanes == 6) share<1>(t, ih, role, k, sh);
                else share<N == 6 ? 2 : 1>(t, ih, role, k, sh);
                return;
            }
        }
        particle_weights<N, AT>(a, t, k.w, k.wd);
    }
    template <typename RowFn>
    __device__ __forceinline__ static void eval(const Args& a, long p, bool active, int lanes, int part,
                                                const Weights& k, RowFn rows) {
        if constexpr (N == 6) {
            if (SHARE && lanes == 6)
                return split_eval<N, CT, AT, C, GRAD, 6, G::PS>(a, p, active && part == 0, part, k.w, k.wd, rows);
            if (lanes == 3)
                return split_eval<N, CT, AT, C, GRAD, 3, G::PS>(a, p, active && part == 0, part, k.w, k.wd, rows);
        } else if constexpr (N == 4) {
            if (lanes == 4)
                return split_eval<N, CT, AT, C, GRAD, 4, G::PS>(a, p, active && part == 0, part, k.w, k.wd, rows);
        }
        if (lanes == 2)
            return pair_eval<N, CT, AT, C, GRAD, G::PS>(a, p, active && part == 0, part, k.w, k.wd, rows);
        Partial<AT, C> lo, hi;
        contract_planes<N, CT, AT, C, GRAD, N / 2, true, G::PS>(k.w[0], k.wd[0], k.w, k.wd, rows, lo);
        contract_planes<N, CT, AT, C, GRAD, N / 2, true, G::PS>(
            k.w[0] + N / 2, k.wd[0] + N / 2, k.w, k.wd, [&](int i, int ib) { return rows(N / 2 + i, ib); }, hi);
        if (active) store_sum<AT, C, GRAD>(a, p, lo, hi);
    }
    template <int B>
    __device__ __forceinline__ static void nonfinite(const Args& a, uint32_t count, uint32_t start) {
        nonfinite_eval<AT, C, GRAD, B>(a, count, start);
    }

   private:
    // Weights of a particle on N / PPL lanes.  Axes 1 and 2: all of them, through
    // LDS.  Axis 0: each of k.w[0][i], i < N / 2, is plane i of the lane's half
    // (the lanes that add a half up read the next lanes' values).
    template <int PPL>
    __device__ __forceinline__ static void share(const AT* t, const double* ih, const LaneRole& role, Weights& k,
                                                 Shared* sh) {
        constexpr int SL = N / PPL, H = N / 2;
        const int lane = threadIdx.x & 63;
        auto& slot = sh->pair[threadIdx.x >> 6][lane / SL];
        AT w0[PPL], wd0[PPL];
#pragma unroll
        for (int i = 0; i < PPL; ++i) {
            const int j = role.part * PPL + i;
            AT c[Shared::ROW];
#pragma unroll
            for (int q = 0; q < Shared::ROW; q += 4)
                *reinterpret_cast<f32x4*>(c + q) = *reinterpret_cast<const f32x4*>(&sh->coef[j][q]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                AT w = c[0], wd = c[N];
#pragma unroll
                for (int q = 1; q < N; ++q) w = fused(w, t[d], c[q]);
#pragma unroll
                for (int q = 1; q < N - 1; ++q) wd = fused(wd, t[d], c[N + q]);
                wd *= AT(ih[d]);
                if (d == 0) {
                    w0[i] = w;
                    wd0[i] = wd;
                } else {
                    slot[d - 1][j][0] = w;
                    slot[d - 1][j][1] = wd;
                }
            }
        }
#pragma unroll
        for (int d = 1; d < 3; ++d)
#pragma unroll
            for (int j = 0; j < N; j += 2) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(&slot[d - 1][j][0]);
                k.w[d][j] = v[0];
                k.wd[d][j] = v[1];
                k.w[d][j + 1] = v[2];
                k.wd[d][j + 1] = v[3];
            }
        // axis 0: planes of the half, in order
        if constexpr (SL == 4) {
            k.w[0][0] = w0[0];
            k.wd[0][0] = wd0[0];
            k.w[0][1] = quad_lane<QUAD_XOR1>(w0[0]);
            k.wd[0][1] = quad_lane<QUAD_XOR1>(wd0[0]);
        } else if constexpr (SL == 6) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                k.w[0][i] = i == 0 ? w0[0] : __shfl(w0[0], (lane + i) & 63, 64);
                k.wd[0][i] = i == 0 ? wd0[0] : __shfl(wd0[0], (lane + i) & 63, 64);
            }
        } else {
            // parts 0 | 1 | 2 hold planes 0 1 | 2 3 | 4 5
            const bool upper = role.part == 2;
            const AT nw = __shfl(w0[0], (lane + 1) & 63, 64), nd = __shfl(wd0[0], (lane + 1) & 63, 64);
            const AT pw = __shfl(w0[PPL - 1], (lane + 63) & 63, 64), pd = __shfl(wd0[PPL - 1], (lane + 63) & 63, 64);
            k.w[0][0] = upper ? pw : w0[0];
            k.wd[0][0] = upper ? pd : wd0[0];
            k.w[0][1] = upper ? w0[0] : w0[PPL - 1];
            k.wd[0][1] = upper ? wd0[0] : wd0[PPL - 1];
            k.w[0][H - 1] = upper ? w0[PPL - 1] : nw;
            k.wd[0][H - 1] = upper ? wd0[PPL - 1] : nd;
        }
#pragma unroll
        for (int i = H; i < N; ++i) {
            k.w[0][i] = k.w[0][i - H];
            k.wd[0][i] = k.wd[0][i - H];
        }
    }
};

// LDS of a persistent workgroup.
template <typename K>
constexpr int tile_lds_bytes() {
    return K::G::SLOTS * 16;
}

// A persistent workgroup of B threads (W wavefronts) of a tiled kernel K: for each
// work item the block of its tile is filled into LDS, then its particles are
// contracted from there.  args_of(tag, a) sets a to the arguments of the items'
// field.  Every thread of the workgroup calls this.
//
// What bounds it is latency, not a rate: at 512^3, order 6, FP32, 5 * 10^6
// particles (1.36 ms, five workgroups' worth of LDS a CU) the contraction alone
// takes 0.87 ms, without the block copies it is 0.99 ms, without the stores 1.25 ms,
// and the vector units are 38 % busy, LDS 35 %.  So a row of four tiles along
// axis 0 is one workgroup's (tile_key), whose block slides and copies 8 of 13
// planes only; a particle's planes are dealt to several lanes and its weights
// formed once (SharedWeights); and items and particle records are requested one
// item ahead.  Against blocks copied whole and lanes that each form all weights:
// 512^3, FP32 order 6, 10^7 clustered particles 2125 -> 1981 us; 256^3, 10^6: order
// 6 231 -> 217, order 4 unchanged at 164.  Half-height blocks with the next planes
// copied during the contraction took 2106 instead of 1405 us, results stored one
// item late 1412 instead of 1364.
template <typename K, int B, typename ArgsOf>
__device__ __forceinline__ void tiled_gather(ArgsOf args_of, const ItemSource& src, bool spread, u32x4* lds,
                                             typename K::Shared* shared, uint32_t* sh) {
    using CT = typename K::CT;
    using AT = typename K::AT;
    using G = typename K::G;
    constexpr int N = K::N, C = K::C, T = K::T, W = B / 64;
    static_assert(sizeof(CT) != 2 || bf16_rows_fit<N, C, T, G::LROW>(), "BF16 row reads would leave the LDS row");
    const CT* tile = reinterpret_cast<const CT*>(lds);
    ItemStream<B> stream;
    u32x4 it;
    if (!stream.begin(src, sh, spread && gridDim.x >= ITEM_RANGES, it)) {
        item_take_end(src.ctl);
        return;
    }
    // particles of one round of an item
    struct Round {
        RawParticle<AT> raw;
        uint32_t p;
        bool active;
    };
    typename K::Args a;
    uint32_t tag = it.w;
    args_of(tag, a);
    K::init(a, shared);
    uint32_t off[plane_steps<G>()];
    plane_offsets<CT, C, G>(a.pitch2, off);
    auto fetch = [&](const u32x4& item, int lanes, uint32_t j0, Round& r) {
        const LaneRole role = lane_role(lanes);
        const uint32_t j = j0 + role.j;
        r.active = j < item.z && role.ok;
        const uint32_t jj = item.y + (r.active ? j : 0u);
        r.p = a.perm[jj];
        r.raw.load(a.binned, long(jj));
    };
    BlockRing<G, T> ring;
    int lanes = K::template lanes<W>(it.z);
    Round r;
    fetch(it, lanes, 0, r);
    for (;;) {
        const int o0 = int(it.x >> 20), o1 = int((it.x >> 10) & 1023u), o2 = int(it.x & 1023u);
        if (it.x != NO_CELL) {
            const int i0 = ring.advance(it.x);
            if (i0 < G::R0)
                block_dma<N, CT, C, G, T, B>(a.grid, a.n0, a.n1, a.P1, a.pitch2, o0, o1, o2, ring, i0, off, lds);
        }
        // everything that has been requested (the last results have gone out
        // meanwhile)
        wait_loads();
        r.raw.settle(r.p);
        stream.settle();
        stream.publish();
        lds_barrier();
        stream.step();
        // the next item's first particles, on their way during the contraction
        // (not across fields: their arguments are not here yet)
        u32x4 nit;
        bool known = stream.next(nit);
        int nlanes = 1;
        Round nr;
        const bool ahead = known && nit.w == tag;
        if (ahead) {
            nlanes = K::template lanes<W>(nit.z);
            fetch(nit, nlanes, 0, nr);
        }
        if (it.x == NO_CELL) {
            K::template nonfinite<B>(a, it.z, it.y);
        } else {
            const LaneRole role = lane_role(lanes);
            const uint32_t first = __builtin_amdgcn_readfirstlane(role.j);
            for (uint32_t j0 = 0;;) {
                Round r2;
                const bool again = lanes == 1 && j0 + uint32_t(B) < it.z;
                if (again) fetch(it, 1, j0 + uint32_t(B), r2);
                // a wavefront without any particle skips the round (uniform);
                // inside a working one, lanes past the end evaluate the
                // item's first particle and store nothing
                if (j0 + first < it.z) {
                    int cell[3];
                    typename K::Weights wts;
                    K::setup(a, r.raw, lanes, role, cell, wts, shared);
                    // row (ia, ib) of the particle's stencil
                    const CT* base = tile + (cell[1] - o1) * G::LROW + (cell[2] - o2) * G::PS;
                    const int c0 = ring.s + cell[0] - o0;
                    auto rows = [base, c0](int ia, int ib) {
                        return base + BlockRing<G, T>::wrap(c0 + ia) * (G::PLANE * G::VEC) + ib * G::LROW;
                    };
                    K::eval(a, long(r.p), r.active, lanes, role.part, wts, rows);
                }
                if (!again) break;
                j0 += uint32_t(B);
                r = r2;
            }
        }
        lds_barrier();   // every LDS read done before planes are replaced
        if (!known) known = stream.next_wait(nit);
        if (!known) break;
        if (!ahead) {
            if (nit.w != tag) {
                tag = nit.w;
                args_of(tag, a);
                plane_offsets<CT, C, G>(a.pitch2, off);
                ring.held = NO_CELL;
            }
            nlanes = K::template lanes<W>(nit.z);
            fetch(nit, nlanes, 0, nr);
        }
        it = nit;
        lanes = nlanes;
        r = nr;
    }
    item_take_end(src.ctl);
}

}  // namespace bsi
