// Internal: a workgroup barrier for LDS traffic alone.
#pragma once

#include <hip/hip_runtime.h>

namespace dmas {

// The workgroup's LDS accesses before it are seen after it; its global loads and
// stores in flight (the next samples, the last outputs) are not waited for.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace dmas
