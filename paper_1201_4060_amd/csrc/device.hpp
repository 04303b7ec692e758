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

}  // namespace bsi
