// Device helpers of more than one kernel file.
#pragma once

#include <hip/hip_runtime.h>

namespace aim {

// LDS values that the lanes of one wave (or of a group within it) exchange: order, no barrier
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace aim
