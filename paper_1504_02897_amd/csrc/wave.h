// Device helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace ddi {

// LDS barrier within a wave: LDS operations of a wave complete in order; the fences keep the compiler from
// moving them across.
__device__ __forceinline__ void lds_sync_wave() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace ddi
