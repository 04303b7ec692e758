// Evaluation on the GPU: position -> cell/offset, binning by tiles, and the
// per-particle gather + tensor contraction (Sections 2, 3, 5; Table 1).
#include <algorithm>

#include "gather.hpp"

namespace bsi {

__global__ void k_debug_cells(CellArgs a, int32_t* cell, double* t) {
    const long p = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (p >= a.P) return;
    const int n[3] = {a.n0, a.n1, a.n2};
    const double ih[3] = {a.ih0, a.ih1, a.ih2};
    int c[3];
    double tt[3];
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) ok = cell_of(a.pos[3 * p + d], ih[d], n[d], c[d], tt[d]) && ok;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        cell[3 * p + d] = ok ? c[d] : -1;
        t[3 * p + d] = ok ? tt[d] : __builtin_nan("");
    }
}

// ---------------------------------------------------------------- binning ---

// Key of a particle: that of its sort tile (tile_key), or nbuckets_finite for a
// non-finite position; its coarse range is key >> shift.
struct TileKey {
    CellArgs a;
    int tile;
    uint32_t nbuckets_finite;
    int shift;
    struct Slot {
        double x[3];
        uint32_t local;
    };
    __device__ __forceinline__ bool fetch(long p, Slot& s) const {
        s.local = uint32_t(p);
        s.x[0] = a.pos[3 * p];
        s.x[1] = a.pos[3 * p + 1];
        s.x[2] = a.pos[3 * p + 2];
        return true;
    }
    __device__ __forceinline__ void place(const Slot& s, GrpPlace& pl) const {
        const int n[3] = {a.n0, a.n1, a.n2};
        const double ih[3] = {a.ih0, a.ih1, a.ih2};
        pl.ok = locate<double>(s.x, n, ih, pl.cell, pl.t);
        pl.key = nbuckets_finite;
        if (pl.ok) {
            const uint32_t T = uint32_t(tile);
            pl.key = tile_key(uint32_t(pl.cell[0]) / T, uint32_t(pl.cell[1]) / T, uint32_t(pl.cell[2]) / T);
        }
        pl.coarse = pl.key >> shift;
    }
};

// The binning read back as one table over all tiles in Morton order (bsi_debug_bins),
// from what a gather reads: chunk descriptors, work items, binned particles.

// Bucket of an item in the table of nb buckets (the last one: no cell).
__device__ __forceinline__ uint32_t item_bucket(const u32x4& it, uint32_t tile, uint32_t nb) {
    if (it.x == NO_CELL) return nb - 1;
    return (spread3((it.x >> 20) / tile) << 2) | (spread3(((it.x >> 10) & 1023u) / tile) << 1) |
           spread3((it.x & 1023u) / tile);
}

// One workgroup per chunk: the items' particles into their buckets' counts.
__global__ __launch_bounds__(256) void k_table_count(ItemSource src, uint32_t tile, uint32_t nb,
                                                    uint32_t* __restrict__ count) {
    if (blockIdx.x >= *src.g1) return;
    const u32x4 d = src.desc[blockIdx.x];
    for (uint32_t i = threadIdx.x; i < d.z; i += 256) {
        const u32x4 it = src.items[d.w + i];
        const uint32_t b = item_bucket(it, tile, nb);
        if (b < nb) atomicAdd(&count[b], it.z);
    }
}

// One workgroup: counts to hist, their exclusive scan to offs and, as cursors, to count.
__global__ __launch_bounds__(1024) void k_table_offsets(uint32_t nb, uint32_t* __restrict__ count,
                                                       uint32_t* __restrict__ hist, uint32_t* __restrict__ offs) {
    __shared__ uint32_t sh[1024 / 64];
    uint32_t before = 0;
    for (uint32_t k0 = 0; k0 < nb; k0 += 1024) {
        const uint32_t k = k0 + threadIdx.x;
        const uint32_t v = k < nb ? count[k] : 0u;
        uint32_t total;
        const uint32_t at = before + block_scan<1024>(v, sh, &total);
        if (k < nb) {
            hist[k] = v;
            offs[k] = at;
            count[k] = at;
        }
        before += total;
    }
}

// One wavefront per chunk: the items' particles to their buckets' slots, with the
// position that the binned particle stands for: an FP64 one's own, for an FP32
// record that of the particle it names if the record is that particle's (else NaN).
template <typename AT>
__global__ __launch_bounds__(64) void k_table_scatter(ItemSource src, CellArgs a, uint32_t tile, uint32_t nb,
                                                      const void* __restrict__ binned,
                                                      const uint32_t* __restrict__ perm,
                                                      uint32_t* __restrict__ cursor, uint32_t* __restrict__ perm_out,
                                                      double* __restrict__ pos_sorted) {
    if (blockIdx.x >= *src.g1) return;
    const u32x4 d = src.desc[blockIdx.x];
    for (uint32_t i = 0; i < d.z; ++i) {
        const u32x4 it = src.items[d.w + i];
        const uint32_t b = item_bucket(it, tile, nb);
        const uint32_t at =
            __builtin_amdgcn_readfirstlane(threadIdx.x == 0 && b < nb ? atomicAdd(&cursor[b], it.z) : 0u);
        for (uint32_t j = threadIdx.x; j < it.z; j += 64) {
            if (b >= nb || long(at) + j >= a.P || long(it.y) + j >= a.P) continue;
            const uint32_t p = perm[it.y + j];
            perm_out[at + j] = p;
            RawParticle<AT> raw;
            raw.load(binned, long(it.y) + j);
            double x[3] = {__builtin_nan(""), __builtin_nan(""), __builtin_nan("")};
            if constexpr (sizeof(AT) == 8) {
                for (int k = 0; k < 3; ++k) x[k] = raw.x[k];
            } else if (long(p) < a.P) {
                const int n[3] = {a.n0, a.n1, a.n2};
                const double ih[3] = {a.ih0, a.ih1, a.ih2};
                const double* y = a.pos + 3 * long(p);
                int cell[3];
                AT t[3];
                const bool ok = locate<AT>(y, n, ih, cell, t);
                bool same = raw.r.w == (ok ? pack_cell(cell) : NO_CELL);
                for (int k = 0; k < 3 && ok; ++k) same = same && raw.r[k] == __float_as_uint(t[k]);
                for (int k = 0; k < 3 && same; ++k) x[k] = y[k];
            }
            for (int k = 0; k < 3; ++k) pos_sorted[3 * (long(at) + j) + k] = x[k];
        }
    }
}

// ----------------------------------------------------------------- gather ---

// Direct variant: one thread per particle.
template <int N, typename CT, int C, bool GRAD>
__global__ __launch_bounds__(256) void k_gather(GatherArgs a) {
    const long j = logical_block(a.xcd_remap) * blockDim.x + threadIdx.x;
    if (j >= a.P) return;
    direct_eval<N, CT, C, GRAD>(a, j);
}

// The same with N lanes per particle (orders 4 and 6), one wavefront a workgroup.
template <int N, typename CT, int C, bool GRAD>
__global__ __launch_bounds__(64) void k_gather_split(GatherArgs a) {
    __shared__ __align__(16) SplitSlots<N, typename Acc<CT>::type> slots;
    direct_split_eval<N, CT, C, GRAD>(a, long(logical_block(a.xcd_remap)) * (64 / N), slots);
}

// Wavefronts per SIMD that a tiled instance is compiled for: as many as its
// registers allow without spilling (its LDS blocks may allow fewer).
template <int N, typename CT, int C>
constexpr int tiled_waves() {
    if (sizeof(CT) == 8) return N == 6 || C == 3 ? 1 : 2;
    return N < 6 && C == 1 ? 3 : 2;
}

// LDS-tiled variant: persistent workgroups of B threads evaluate work items
// (pieces of tiles of T^3 cells, k_grp_fine), with xcd_remap those of the
// range blockIdx % ITEM_RANGES first (workgroups are dispatched to the XCDs in
// turn).
template <int N, typename CT, int C, bool GRAD, int T, int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(tiled_waves<N, CT, C>()))) void
k_gather_tiled(GatherArgs a) {
    using K = ValueGather<N, CT, C, GRAD, T, B / 64>;
    __shared__ u32x4 tile_v[tile_lds_bytes<K>() / 16];
    __shared__ __align__(16) typename K::Shared shared;
    __shared__ uint32_t taken[3];
    tiled_gather<K, B>([&](uint32_t, GatherArgs& x) { x = a; }, a.src,
                       a.xcd_remap != 0, tile_v, &shared, taken);
}

// ------------------------------------------------------------- launchers ---

namespace {

CellArgs cell_args(const bsi_field* f, const double* pos, long P) {
    CellArgs a;
    a.pos = pos;
    a.P = P;
    a.n0 = f->n[0];
    a.n1 = f->n[1];
    a.n2 = f->n[2];
    a.ih0 = f->inv_h[0];
    a.ih1 = f->inv_h[1];
    a.ih2 = f->inv_h[2];
    return a;
}

// Several lanes per particle (k_gather_split) or one (k_gather).  Unbinned: several
// while the particles do not fill the chip's wavefronts one lane each (64^3 FP32
// order 6: 10^4 particles 22 against 32 us, 2 * 10^4 27 / 33, 4 * 10^4 37 / 35; 256^3
// BF16 order 6, whose rows are read four bytes at a time: 2 * 10^4 23 / 28, 2.5 * 10^4
// 29 / 28, 3 * 10^4 34 / 29).
// Binned: several for a sparse cloud, whose particles share little in the cache
// (whole evaluations; 1024^3 BF16 scalar, 4 * 10^6: 1502 / 2070 us, 256^3 FP32 order
// 6, 1.6 * 10^5: 122 / 167; from one particle in eight cells on one lane does with
// fewer instructions: 128^3 FP32 scalar, 10^6: 178 / 158), but one again for the
// largest stencils below one particle in 256 cells, bound by memory pages (512^3
// FP32 order 6, 3.2 * 10^5: 421 / 379, 256^3, 8 * 10^4: 88 / 113; 256^3 FP64 order 4,
// 6 * 10^4: 72 / 66).
bool split_lanes(const bsi_field* f, long P, bool binned) {
    const int stencil = f->N * f->N * f->N * f->C;
    if (!binned) return P < (f->desc.coef == BSI_BF16 && stencil >= 512 ? 24576 : 32768);
    const double dens = double(P) / (double(f->n[0]) * f->n[1] * f->n[2]);
    const bool large = stencil >= (f->desc.coef == BSI_F64 ? 192 : 512);
    return dens < 1.0 / 8 && (!large || dens >= 1.0 / 256);
}

template <int N, typename CT, int C>
void launch_gather_t(const GatherArgs& ga, bool grad, bool split, unsigned nb, unsigned block, hipStream_t s) {
    if constexpr (N > 2) {
        if (split) {
            const unsigned ns = unsigned((ga.P + 64 / N - 1) / (64 / N));
            if (grad) hipLaunchKernelGGL((k_gather_split<N, CT, C, true>), dim3(ns), dim3(64), 0, s, ga);
            else hipLaunchKernelGGL((k_gather_split<N, CT, C, false>), dim3(ns), dim3(64), 0, s, ga);
            return;
        }
    }
    if (grad)
        hipLaunchKernelGGL((k_gather<N, CT, C, true>), dim3(nb), dim3(block), 0, s, ga);
    else
        hipLaunchKernelGGL((k_gather<N, CT, C, false>), dim3(nb), dim3(block), 0, s, ga);
}

template <typename CT>
void launch_gather_ct(int N, int C, const GatherArgs& ga, bool grad, bool split, unsigned nb, unsigned block,
                      hipStream_t s) {
    if (N == 2) {
        if (C == 1) launch_gather_t<2, CT, 1>(ga, grad, split, nb, block, s);
        else launch_gather_t<2, CT, 3>(ga, grad, split, nb, block, s);
    } else if (N == 4) {
        if (C == 1) launch_gather_t<4, CT, 1>(ga, grad, split, nb, block, s);
        else launch_gather_t<4, CT, 3>(ga, grad, split, nb, block, s);
    } else {
        if (C == 1) launch_gather_t<6, CT, 1>(ga, grad, split, nb, block, s);
        else launch_gather_t<6, CT, 3>(ga, grad, split, nb, block, s);
    }
}

constexpr int TILE_LDS_LIMIT = 64 * 1024;  // static LDS per workgroup

template <int N, typename CT, int C, int T>
constexpr bool tile_ok() {
    return TileGeom<N, CT, C, T>::BYTES <= TILE_LDS_LIMIT && TileGeom<N, CT, C, T>::ALIGNED;
}

// Threads per workgroup: 64 for small blocks, 128 where at most five blocks of
// 64 would fit a CU's LDS (5 * 10^6 particles at 512^3, FP32 order 6: 1382 us,
// with 64 threads 1443; BF16, 14 KB blocks: 64 threads 1665, 128 1924; FP32
// order 4, 21 KB: 165 and 171 at 256^3), 256 for blocks that fill the LDS budget.
// FP64 order 6 instances hold up to 376 registers, one wavefront a SIMD: 128, so that
// two workgroups share a CU and one copies while the other evaluates (300007
// particles at 192 x 128 x 256: 270 us; with 64 threads 287, with 256 364).  FP64
// scalars and below order 6, whose blocks let four workgroups or more share a CU: 64
// (10^6 particles at 256^3, order 4: 229 us, with 128 threads 261, clustered 266 / 298, scalar
// order 6 168 / 262; for the dense tiles of 64^3 order 4 it is the other way round, 105 / 94).
template <int N, typename CT, int C, int T>
constexpr int tile_block() {
    if (sizeof(CT) == 8) return N == 6 && C == 3 ? 128 : 64;
    return TileGeom<N, CT, C, T>::SLOTS >= 3072 ? 256 : TileGeom<N, CT, C, T>::SLOTS >= 2048 ? 128 : 64;
}

// The tiled gather runs as many workgroups as can be resident at once (its
// occupancy, asked once per instance, on every CU).
template <int N, typename CT, int C, bool GRAD, int T, int B>
void launch_tiled_kernel(const GatherArgs& ga, int num_cus, hipStream_t s) {
    auto k = k_gather_tiled<N, CT, C, GRAD, T, B>;
    static unsigned nb = 0;
    static std::once_flag once;
    std::call_once(once, [&] {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k, B, 0) != hipSuccess || v < 1) v = 1;
        nb = unsigned(v);
    });
    hipLaunchKernelGGL(k, dim3(nb * unsigned(std::max(num_cus, 1))), dim3(B), 0, s, ga);
}

template <int N, typename CT, int C, int T>
bool launch_tiled_T(const GatherArgs& ga, bool grad, bool wide, int num_cus, hipStream_t s) {
    if constexpr (!tile_ok<N, CT, C, T>()) {
        return false;
    } else {
        constexpr int B = tile_block<N, CT, C, T>();
        if constexpr (T == 8 && B < 256) {
            // dense 8^3 tiles: four wavefronts share one LDS block
            if (wide) {
                if (grad) launch_tiled_kernel<N, CT, C, true, T, 256>(ga, num_cus, s);
                else launch_tiled_kernel<N, CT, C, false, T, 256>(ga, num_cus, s);
                return true;
            }
        }
        if (grad) launch_tiled_kernel<N, CT, C, true, T, B>(ga, num_cus, s);
        else launch_tiled_kernel<N, CT, C, false, T, B>(ga, num_cus, s);
        return true;
    }
}

// threads per workgroup of the tiled gather for this field and tile (0 if no
// tiled instance)
template <int N, typename CT, int C, int T>
constexpr int tiled_block_T(bool wide) {
    if constexpr (!tile_ok<N, CT, C, T>()) return 0;
    else return (T == 8 && tile_block<N, CT, C, T>() < 256 && wide) ? 256 : tile_block<N, CT, C, T>();
}

template <int N, typename CT, int C>
bool launch_tiled_c(int T, const GatherArgs& ga, bool grad, bool wide, int num_cus, hipStream_t s) {
    switch (T) {
        case 4: return launch_tiled_T<N, CT, C, 4>(ga, grad, wide, num_cus, s);
        case 6: return launch_tiled_T<N, CT, C, 6>(ga, grad, wide, num_cus, s);
        case 8: return launch_tiled_T<N, CT, C, 8>(ga, grad, wide, num_cus, s);
        case 12: return launch_tiled_T<N, CT, C, 12>(ga, grad, wide, num_cus, s);
        case 16: return launch_tiled_T<N, CT, C, 16>(ga, grad, wide, num_cus, s);
        default: return false;
    }
}

template <typename CT>
bool launch_tiled_ct(int N, int C, int T, const GatherArgs& ga, bool grad, bool wide, int num_cus,
                     hipStream_t s) {
    if (N == 2) {   // linear: 8^3-cell tiles only
        if (T != 8) return false;
        return C == 1 ? launch_tiled_T<2, CT, 1, 8>(ga, grad, wide, num_cus, s)
                      : launch_tiled_T<2, CT, 3, 8>(ga, grad, wide, num_cus, s);
    }
    if (N == 4)
        return C == 1 ? launch_tiled_c<4, CT, 1>(T, ga, grad, wide, num_cus, s)
                      : launch_tiled_c<4, CT, 3>(T, ga, grad, wide, num_cus, s);
    return C == 1 ? launch_tiled_c<6, CT, 1>(T, ga, grad, wide, num_cus, s)
                  : launch_tiled_c<6, CT, 3>(T, ga, grad, wide, num_cus, s);
}

template <int N, typename CT, int C>
int tiled_block_c(int T, bool wide) {
    switch (T) {
        case 4: return tiled_block_T<N, CT, C, 4>(wide);
        case 6: return tiled_block_T<N, CT, C, 6>(wide);
        case 8: return tiled_block_T<N, CT, C, 8>(wide);
        case 12: return tiled_block_T<N, CT, C, 12>(wide);
        case 16: return tiled_block_T<N, CT, C, 16>(wide);
        default: return 0;
    }
}

template <typename CT>
int tiled_block_ct(int N, int C, int T, bool wide) {
    if (N == 2) {
        if (T != 8) return 0;
        return C == 1 ? tiled_block_T<2, CT, 1, 8>(wide) : tiled_block_T<2, CT, 3, 8>(wide);
    }
    if (N == 4) return C == 1 ? tiled_block_c<4, CT, 1>(T, wide) : tiled_block_c<4, CT, 3>(T, wide);
    return C == 1 ? tiled_block_c<6, CT, 1>(T, wide) : tiled_block_c<6, CT, 3>(T, wide);
}

template <int N, typename CT, int C>
bool tile_ok_rt(int T) {
    switch (T) {
        case 4: return tile_ok<N, CT, C, 4>();
        case 6: return tile_ok<N, CT, C, 6>();
        case 8: return tile_ok<N, CT, C, 8>();
        case 12: return tile_ok<N, CT, C, 12>();
        case 16: return tile_ok<N, CT, C, 16>();
        default: return false;
    }
}

template <typename CT>
bool tile_ok_ct(int N, int C, int T) {
    if (N == 2) return T == 8 && (C == 1 ? tile_ok<2, CT, 1, 8>() : tile_ok<2, CT, 3, 8>());
    if (N == 4) return C == 1 ? tile_ok_rt<4, CT, 1>(T) : tile_ok_rt<4, CT, 3>(T);
    return C == 1 ? tile_ok_rt<6, CT, 1>(T) : tile_ok_rt<6, CT, 3>(T);
}

}  // namespace

size_t bin_bucket_count(const bsi_field* f, int tile) {
    int bits = 0;
    for (int d = 0; d < 3; ++d) {
        const int nt = (f->n[d] + tile - 1) / tile;
        int b = 0;
        while ((1 << b) < nt) ++b;
        bits = std::max(bits, b);
    }
    return size_t(1) << (3 * bits);
}

size_t bin_key_count(const bsi_field* f, int tile) {
    // whole bricks of 4^3 tiles, as many along every axis (a power of two)
    int bits = 0;
    for (int d = 0; d < 3; ++d)
        while (((4 * tile) << bits) < f->n[d]) ++bits;
    return size_t(64) << (3 * bits);
}

// At most 2^24 + 1 keys (effective_tile).
static GrpPlan bin_plan(size_t keys, long P, int* shift) {
    const uint64_t nb = keys + 1;
    *shift = grp_shift(nb, P);
    const uint32_t ncoarse = uint32_t((nb + (uint64_t(1) << *shift) - 1) >> *shift);
    return grp_plan(P, uint32_t(P), uint32_t(nb), ncoarse, uint32_t(std::min<uint64_t>(nb, uint64_t(1) << *shift)));
}

// Workspace of a binned evaluation (16-byte aligned): the grouping scratch,
// the binned particles (16 bytes each, FP64 fields 24), the permutation, and
// with work items of at most `ichunk` particles (0: none) the items and their
// control words.
BinLayout bin_layout(const bsi_field* f, long P, int tile, uint32_t ichunk) {
    int shift = 0;
    const GrpPlan g = bin_plan(bin_key_count(f, tile), P, &shift);
    BinLayout l;
    l.ichunk = ichunk;
    l.grp = 0;
    l.binned = (grp_scratch_words(g) * sizeof(uint32_t) + 15) / 16 * 16;
    l.perm = l.binned + size_t(P) * (f->desc.coef == BSI_F64 ? 24 : 16);
    l.items = (l.perm + size_t(P) * sizeof(uint32_t) + 15) / 16 * 16;
    l.ctl = l.items + (ichunk ? grp_item_cap(g, ichunk) * sizeof(u32x4) : 0);
    l.bytes = l.ctl + (ichunk ? ITEM_CTL_WORDS * sizeof(uint32_t) : 0);
    return l;
}

BinArrays bin_arrays(const bsi_field* f, long P, int tile, const BinLayout& l, void* ws) {
    char* w = static_cast<char*>(ws);
    int shift = 0;
    const GrpPlan g = bin_plan(bin_key_count(f, tile), P, &shift);
    const GrpBuffers gb = grp_buffers(g, reinterpret_cast<uint32_t*>(w + l.grp));
    BinArrays b;
    b.units_log2 = l.ichunk ? item_units_log2(g, l.ichunk, ITEM_UNITS, f->N <= 4) : 0;
    b.desc = gb.desc;
    b.nchunks = gb.nchunks;
    b.binned = w + l.binned;
    b.perm = reinterpret_cast<uint32_t*>(w + l.perm);
    b.items = l.ichunk ? w + l.items : nullptr;
    b.ctl = l.ichunk ? reinterpret_cast<uint32_t*>(w + l.ctl) : nullptr;
    return b;
}

bsi_status bin_run(bsi_field* f, const double* pos, long P, int tile, const BinLayout& l, void* ws, hipStream_t s) {
    const size_t nbf = bin_key_count(f, tile);
    int shift = 0;
    const GrpPlan g = bin_plan(nbf, P, &shift);
    const GrpBuffers gb = grp_buffers(g, reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + l.grp));
    const BinArrays b = bin_arrays(f, P, tile, l, ws);
    const TileKey mk{cell_args(f, pos, P), tile, uint32_t(nbf), shift};
    const ShiftCoarse cm{shift, uint32_t(nbf + 1)};
    const OneField ls{b.ctl != nullptr, uint32_t(tile), uint32_t(nbf)};
    const uint32_t ichunk = l.ichunk ? l.ichunk : GRP_CHUNK;
    {
        StageTimer tm(f->ctx, "bin_count", s);
        grp_count(mk, g, gb, b.ctl, b.ctl ? ITEM_CTL_WORDS : 0, s);
    }
    {
        StageTimer tm(f->ctx, "bin_scan", s);
        grp_scan(g, gb, s);
    }
    {
        StageTimer tm(f->ctx, "bin_scatter", s);
        u32x4* items = static_cast<u32x4*>(b.items);
        if (f->desc.coef == BSI_F64) grp_scatter<false>(mk, cm, ls, g, gb, ichunk, b.perm, b.binned, items, s);
        else grp_scatter<true>(mk, cm, ls, g, gb, ichunk, b.perm, b.binned, items, s);
    }
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

bool tiled_supported(const bsi_field* f, int tile) {
    // Hermite fields (two stored entries per cell and axis) use the direct gather
    if (f->cs != 1) return false;
    if (f->desc.coef == BSI_F64) return tile_ok_ct<double>(f->N, f->C, tile);
    if (f->desc.coef == BSI_F32) return tile_ok_ct<float>(f->N, f->C, tile);
    return tile_ok_ct<uint16_t>(f->N, f->C, tile);
}

// Sort tile actually used: at least n/256 cells per tile edge, so that the
// bucket table has at most 2^24 entries.
static int effective_tile(const bsi_field* f, const bsi_eval_config& cfg) {
    if (cfg.sort_tile <= 0) return 0;
    const int nmax = std::max(f->n[0], std::max(f->n[1], f->n[2]));
    return std::max(cfg.sort_tile, (nmax + 255) / 256);
}

// Threads per workgroup of the tiled gather for field f, tile and config (0:
// no tiled instance, the direct gather runs).
static int tiled_block(const bsi_field* f, int tile, const bsi_eval_config& cfg) {
    if (tile == 0 || cfg.variant != 0 || !tiled_supported(f, tile)) return 0;
    const bool wide = cfg.tile_block == 256;
    if (f->desc.coef == BSI_F64) return tiled_block_ct<double>(f->N, f->C, tile, wide);
    if (f->desc.coef == BSI_F32) return tiled_block_ct<float>(f->N, f->C, tile, wide);
    return tiled_block_ct<uint16_t>(f->N, f->C, tile, wide);
}

// Particles per work item of the tiled gather (0: the direct gather runs).
static uint32_t item_chunk(const bsi_field* f, int tile, const bsi_eval_config& cfg) {
    return uint32_t(tiled_block(f, tile, cfg)) * uint32_t(cfg.item_rounds > 0 ? cfg.item_rounds : 4);
}

size_t eval_ws_bytes(const bsi_field* f, int64_t P, const bsi_eval_config& cfg) {
    const int tile = effective_tile(f, cfg);
    if (tile == 0 || P == 0) return 0;
    return bin_layout(f, P, tile, item_chunk(f, tile, cfg)).bytes;
}

// The most that any P' <= P takes.  A coarse range holds twice the keys for particle
// counts below a step of grp_shift, and more items are reserved for its chunks, so
// fewer particles can take a little more; between two steps every part of the
// workspace grows with P', so the counts just below the steps and P itself tell.
size_t eval_ws_capacity(const bsi_field* f, int64_t P, const bsi_eval_config& cfg) {
    const int tile = effective_tile(f, cfg);
    if (tile == 0 || P == 0) return 0;
    size_t most = eval_ws_bytes(f, P, cfg);
    const uint64_t nb = bin_key_count(f, tile) + 1;
    for (int s = grp_shift(nb, P) + 1; s <= grp_shift(nb, 1); ++s)
        most = std::max(most, eval_ws_bytes(f, std::min(P, grp_shift_end(nb, s)), cfg));
    return most;
}

bsi_status eval_check_config(const bsi_eval_config& cfg) {
    const int block = cfg.block > 0 ? cfg.block : 256;
    BSI_CHECK(block % 64 == 0 && block >= 64 && block <= 256, BSI_E_INVAL,
              "eval block must be 64, 128, 192 or 256");
    BSI_CHECK(cfg.sort_tile >= 0 && cfg.sort_tile <= 1024, BSI_E_INVAL, "sort_tile out of range");
    BSI_CHECK(cfg.tile_block == 0 || cfg.tile_block == 64 || cfg.tile_block == 256, BSI_E_INVAL,
              "tile_block must be 0, 64 or 256");
    BSI_CHECK(cfg.item_rounds >= 0 && cfg.item_rounds <= 1024, BSI_E_INVAL, "item_rounds must be 0..1024");
    return BSI_OK;
}

// The position-only half of an evaluation: binning and work items into ws
// (nothing without binning).
bsi_status eval_bin_ws(bsi_field* f, const double* pos, int64_t P, const bsi_eval_config& cfg, hipStream_t s,
                       void* ws) {
    const int tile = effective_tile(f, cfg);
    if (P == 0 || tile == 0) return BSI_OK;
    BSI_CHECK(ws != nullptr && reinterpret_cast<uintptr_t>(ws) % 16 == 0, BSI_E_INVAL,
              "binned evaluation needs a 16-byte aligned workspace");
    return bin_run(f, pos, P, tile, bin_layout(f, P, tile, item_chunk(f, tile, cfg)), ws, s);
}

// The gather half: reads the binning eval_bin_ws left in ws for the same
// (pos, P, cfg) and the field's current grid.
bsi_status eval_gather_ws(bsi_field* f, const double* pos, int64_t P, void* u, void* grad,
                          const bsi_eval_config& cfg, hipStream_t s, void* ws) {
    if (P == 0) return BSI_OK;
    const int block = cfg.block > 0 ? cfg.block : 256;
    const int tile = effective_tile(f, cfg);
    GatherArgs ga;
    ga.grid = f->grid;
    ga.pos = pos;
    ga.perm = nullptr;
    ga.binned = nullptr;
    ga.src = ItemSource{};
    if (tile > 0) {
        BSI_CHECK(ws != nullptr && reinterpret_cast<uintptr_t>(ws) % 16 == 0, BSI_E_INVAL,
                  "binned evaluation needs a 16-byte aligned workspace");
        const BinArrays b = bin_arrays(f, P, tile, bin_layout(f, P, tile, item_chunk(f, tile, cfg)), ws);
        ga.perm = b.perm;
        ga.binned = b.binned;
        ga.src = item_source(b);
    }
    ga.u = u;
    ga.grad = grad;
    ga.nonfinite = f->counters;
    ga.P = P;
    ga.n0 = f->n[0];
    ga.n1 = f->n[1];
    ga.n2 = f->n[2];
    ga.P1 = f->P[1];
    ga.pitch2 = f->pitch2;
    ga.ih0 = f->inv_h[0];
    ga.ih1 = f->inv_h[1];
    ga.ih2 = f->inv_h[2];
    ga.xcd_remap = (ga.perm && cfg.xcd_remap) ? 1 : 0;
    ga.basis = f->basis;
    ga.cs = f->cs;
    const bool g = grad != nullptr;
    StageTimer tm(f->ctx, "gather", s);
    if (ga.src.items) {
        bool ok = false;
        // tile_block 256 asks for four wavefronts per 8^3 tile (dense tiles)
        const bool wide = cfg.tile_block == 256;
        const int ncu = f->ctx->num_cus;
        if (f->desc.coef == BSI_F64) ok = launch_tiled_ct<double>(f->N, f->C, tile, ga, g, wide, ncu, s);
        else if (f->desc.coef == BSI_F32) ok = launch_tiled_ct<float>(f->N, f->C, tile, ga, g, wide, ncu, s);
        else ok = launch_tiled_ct<uint16_t>(f->N, f->C, tile, ga, g, wide, ncu, s);
        BSI_CHECK(ok, BSI_E_UNSUPPORTED, "no tiled gather instance for this tile size");
    } else {
        const unsigned nb = unsigned((P + block - 1) / block);
        const bool split = split_lanes(f, long(P), tile > 0);
        if (f->desc.coef == BSI_F64) launch_gather_ct<double>(f->N, f->C, ga, g, split, nb, block, s);
        else if (f->desc.coef == BSI_F32) launch_gather_ct<float>(f->N, f->C, ga, g, split, nb, block, s);
        else launch_gather_ct<uint16_t>(f->N, f->C, ga, g, split, nb, block, s);
    }
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

bsi_status eval_run_ws(bsi_field* f, const double* pos, int64_t P, void* u, void* grad,
                       const bsi_eval_config& cfg, hipStream_t s, void* ws) {
    if (P == 0) return BSI_OK;
    BSI_TRY(eval_check_config(cfg));
    BSI_TRY(eval_bin_ws(f, pos, P, cfg, s, ws));
    return eval_gather_ws(f, pos, P, u, grad, cfg, s, ws);
}

bsi_status eval_run(bsi_field* f, const double* pos, int64_t P, void* u, void* grad,
                    const bsi_eval_config& cfg, hipStream_t s) {
    if (P == 0) return BSI_OK;
    void* ws = nullptr;
    const size_t need = eval_ws_bytes(f, P, cfg);
    if (need) BSI_TRY(get_workspace(f->ctx->eval_ws, s, need, &ws));
    return eval_run_ws(f, pos, P, u, grad, cfg, s, ws);
}

bsi_status debug_cells_run(bsi_field* f, const double* pos, int64_t P, int32_t* cell, double* t,
                           hipStream_t s) {
    if (P == 0) return BSI_OK;
    const CellArgs ca = cell_args(f, pos, P);
    hipLaunchKernelGGL(k_debug_cells, dim3(unsigned((P + 255) / 256)), dim3(256), 0, s, ca, cell, t);
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

bsi_status debug_bins_run(bsi_field* f, const double* pos, int64_t P, int tile, uint32_t* hist, uint32_t* offs,
                          uint32_t* perm, double* pos_sorted, hipStream_t s) {
    const size_t nb = bin_bucket_count(f, tile) + 1;
    if (P == 0) {
        BSI_HIP(hipMemsetAsync(hist, 0, nb * sizeof(uint32_t), s));
        BSI_HIP(hipMemsetAsync(offs, 0, nb * sizeof(uint32_t), s));
        return BSI_OK;
    }
    const BinLayout l = bin_layout(f, long(P), tile, 512u);
    const size_t table = (l.bytes + 15) / 16 * 16;
    void* ws = nullptr;
    BSI_TRY(get_workspace(f->ctx->eval_ws, s, table + nb * sizeof(uint32_t), &ws));
    uint32_t* count = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + table);
    BSI_TRY(bin_run(f, pos, long(P), tile, l, ws, s));
    const BinArrays b = bin_arrays(f, long(P), tile, l, ws);
    const ItemSource src = item_source(b);
    const CellArgs ca = cell_args(f, pos, long(P));
    int shift = 0;
    const unsigned chunks = bin_plan(bin_key_count(f, tile), long(P), &shift).mmax;
    hipLaunchKernelGGL(k_fill_u32, dim3(unsigned(std::min<size_t>((nb + 255) / 256, 4096))), dim3(256), 0, s, count,
                       long(nb), 0u);
    hipLaunchKernelGGL(k_table_count, dim3(chunks), dim3(256), 0, s, src, uint32_t(tile), uint32_t(nb), count);
    hipLaunchKernelGGL(k_table_offsets, dim3(1), dim3(1024), 0, s, uint32_t(nb), count, hist, offs);
    auto scatter = f->desc.coef == BSI_F64 ? k_table_scatter<double> : k_table_scatter<float>;
    hipLaunchKernelGGL(scatter, dim3(chunks), dim3(64), 0, s, src, ca, uint32_t(tile), uint32_t(nb), b.binned, b.perm,
                       count, perm, pos_sorted);
    BSI_HIP(hipGetLastError());
    return BSI_OK;
}

}  // namespace bsi
