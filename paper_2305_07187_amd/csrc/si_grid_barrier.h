// Grid-wide barrier of the resident launches.
#pragma once

#include "si_internal.h"

namespace si {

// Grid-wide barrier of a resident launch, without atomic read-modify-write:
// group g publishes the number of steps it has completed in flags[g] (a
// release store, which also writes this XCD's L2 back), and the first wave
// of every group polls all the flags, one per lane, with plain loads until
// each has reached `step`.  A single acquire fence per group then
// invalidates the stale lines before the next step reads q.  The wait is
// bounded (about 2 s of the 100 MHz real-time counter, and at most 2^26
// polls): a barrier that cannot complete sets *err and every group leaves
// instead of hanging.
__device__ __forceinline__ bool grid_barrier(uint32_t *flags, uint32_t step, int32_t *err) {
  __shared__ int32_t pass;
  const int groups = gridDim.x;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(flags + blockIdx.x, step, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const uint64_t start = __builtin_amdgcn_s_memrealtime();
    int32_t ok = 1;
    uint32_t polls = 0;
    for (;;) {
      bool ready = true;
      for (int g = lane; g < groups; g += 64)
        ready &= __hip_atomic_load(flags + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= step;
      if (__all(ready)) break;
      if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        ok = 0;
        break;
      }
      if (__builtin_amdgcn_s_memrealtime() - start > 200000000ull || ++polls > (1u << 26)) {
        if (lane == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (lane == 0) pass = ok;
  }
  __syncthreads();
  return pass != 0;
}

}  // namespace si
