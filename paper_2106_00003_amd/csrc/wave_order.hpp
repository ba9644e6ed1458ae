// Order between the lanes of a wavefront that share memory in LDS.
#pragma once
#include <hip/hip_runtime.h>

namespace givens {

// Between stores to LDS by a wavefront's lanes and loads of the same places by others of them, or the other way round.  A
// wavefront's LDS operations run in order, so this only holds the compiler to it.
__device__ __forceinline__ void wavefront_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

} // namespace givens
