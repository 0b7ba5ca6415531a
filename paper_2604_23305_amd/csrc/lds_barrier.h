// Workgroup barrier for what is shared in LDS alone: global loads and stores
// stay in flight across it (__syncthreads waits for them).
#pragma once

#include <hip/hip_runtime.h>

namespace gtod {

__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace gtod
