// Ordering inside one wavefront.
#pragma once

#include <hip/hip_runtime.h>

namespace s2w {

// Orders the LDS accesses of one wavefront's lanes (the hardware runs them in issue order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace s2w
