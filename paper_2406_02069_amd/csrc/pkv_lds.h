// Workgroup barrier for kernels whose waves exchange LDS contents only.
#pragma once

#include <hip/hip_runtime.h>

namespace pkv {
namespace {

// Workgroup barrier that orders LDS traffic only.  A full __syncthreads() carries fences over global memory too, and the
// waits the compiler builds for them cover, since memory operations retire in order, the global loads still in flight: a memory
// round trip per use, where only LDS contents change hands.  (Neither kind of barrier waits for the acknowledgement of
// outstanding global stores: where another workgroup is told that data is ready, the storing waves wait for vmcnt(0) themselves.)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace
}  // namespace pkv
