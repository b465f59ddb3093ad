// Data exchange between the workgroups of one cooperative launch.
//
// A workgroup publishes values with agent-scope atomic stores (which pass the
// XCD's own L2) and sets its epoch flag once they have completed; a reader
// takes them with agent-scope atomic loads once every flag has reached the
// epoch.  No fences: an agent-scope acquire would drop the XCD's cached lines
// of everything else, at each exchange.  Among 4 to 62 workgroups an exchange
// takes about 2 us.
//
// Every wait is bounded.  The launch is cooperative, but a long kernel of another
// stream can hold the CUs that some of the workgroups still need, so a wait does
// run out in earnest, and the kernel's caller has to go on without it.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace pdd {

template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by every thread of each of the G workgroups with the same `epoch`,
// one more at each exchange of a launch and above every flag before the first
// one (the flags are cleared, or left by an earlier launch at lower epochs).
// False, for the whole workgroup, once a wait has run out: more than `polls`
// of it failed (0: every wait, at once).  `stop`: a word in LDS, zero before
// the first call.  Workgroup barriers at both ends (also for G = 1).
__device__ __forceinline__ bool grid_exchange(uint32_t* flags, int G, int me, uint32_t epoch, int32_t* stop,
                                              uint32_t polls) {
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (G > 1) {
    if (threadIdx.x == 0) agent_store(flags + me, epoch);
    if (threadIdx.x < 64) {
      const int lane = threadIdx.x;
      uint32_t spins = polls ? 0 : 1;
      for (int q = lane; q - lane < G && spins <= polls; q += 64) {          // uniform trip count
        while (__ballot(q < G && agent_load(flags + (q < G ? q : 0)) < epoch) != 0) {
          __builtin_amdgcn_s_sleep(1);
          if (++spins > polls) break;
        }
      }
      if (spins > polls && lane == 0) *stop = 1;
    }
  }
  __syncthreads();
  return *stop == 0;
}

}  // namespace pdd
