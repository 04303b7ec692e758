// Device helpers shared by the transform and the gather kernels.
#pragma once

namespace bsi {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Barrier for LDS only: orders the wavefront's LDS accesses without waiting for
// outstanding global loads and stores (the next block's loads stay in flight).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// a * b + c with one rounding, written out where the compiler would otherwise
// fuse in one kernel and not in another (products that two methods' weights have
// in common are moved out of the branch between them; the transform's instances).
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

}  // namespace bsi
