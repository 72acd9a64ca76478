#pragma once
#include <hip/hip_runtime.h>

namespace mnnconv {

// LDS writes of this wavefront done, then all wavefronts: loads from global memory stay in flight
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace mnnconv
