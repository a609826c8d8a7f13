// Order of LDS accesses inside a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace hx {

// Order of LDS accesses between the lanes of one wave, whose LDS operations
// execute in order: only the compiler has to keep them so.
__device__ __forceinline__ void lds_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace hx
