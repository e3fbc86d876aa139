// Grid-wide waits of the cooperative kernels (the tail kernel and the core
// kernel): the barrier between two phases and the check-in at entry.
#pragma once

#include "inc.hpp"

namespace gcol {

// Grid-wide barrier.  Workgroups arrive in eight groups (blockIdx.x mod 8,
// each with its own counter bar[kBarGroup + 32 g]); the last of a group
// arrives at the top counter bar[0], and the last of those bumps the
// generation word bar[kBarGen].  Every word sits on its own cache line, so
// arrivals contend eight ways less than on one counter (measured on MI355X:
// 2.8 instead of 7.0 us per barrier at 512 workgroups).  Every array that
// one workgroup writes and another reads within the tail kernel is accessed
// with device-scope loads, stores and atomics, so the barrier needs no cache
// writeback or invalidation: each wavefront waits until its own memory
// operations have completed, and the generation bump is a release.  The
// cooperative launch makes every workgroup co-resident, so a barrier waits
// only for the others to finish their phase; the deadline (wall-clock ticks)
// turns a defect into an error bit instead of a hang.  Returns false (in
// every thread of the workgroup) if it gave up.
__device__ __forceinline__ bool grid_sync(uint32_t* bar, int32_t* err, uint64_t deadline, int32_t* s_ok) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t gen = atomic_load_u32(&bar[kBarGen]);
    const uint32_t G = gridDim.x, g = blockIdx.x & 7u;
    const uint32_t groups = G < 8u ? G : 8u;
    const uint32_t size = G < 8u ? 1u : G / 8u + (g < (G & 7u) ? 1u : 0u);
    uint32_t* gc = &bar[kBarGroup + 32u * g];
    bool last = false;
    if (atomicAdd(gc, 1u) == size - 1u) {
      (void)__hip_atomic_exchange(gc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (atomicAdd(&bar[0], 1u) == groups - 1u) {
        (void)__hip_atomic_exchange(&bar[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&bar[kBarGen], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        last = true;
      }
    }
    int32_t ok = 1;
    if (!last) {
      const uint64_t t0 = static_cast<uint64_t>(wall_clock64());
      while (atomic_load_u32(&bar[kBarGen]) == gen) {
        __builtin_amdgcn_s_sleep(2);
        if (static_cast<uint64_t>(wall_clock64()) - t0 > deadline) {
          atomicOr(err, kErrTailBarrier);
          ok = 0;
          break;
        }
      }
    }
    *s_ok = ok;
  }
  __syncthreads();
  return *s_ok != 0;
}

// Entry check-in of the tail kernel.  Its grid barriers need every workgroup
// resident at once, which the cooperative launch provides only while no
// other kernel fills the device.  So before writing anything, every
// workgroup arrives and waits until either all gridDim.x workgroups have
// arrived (then all are resident: none leaves before the decision) or
// `ticks` have passed.  The decision is one compare-and-swap on a state word
// (the last arrival sets GO, a workgroup whose wait ran out sets ABORT), so
// every workgroup takes the same one, including those that start after it.
// On ABORT the launch changes nothing and the host runs the rounds as
// per-round launches.
constexpr uint32_t kCheckinGo = 1u, kCheckinAbort = 2u;

__device__ __forceinline__ bool tail_checkin(uint32_t* arrived, uint32_t* state, int32_t* err, uint64_t ticks,
                                             int32_t* s_ok) {
  if (threadIdx.x == 0) {
    if (atomicAdd(arrived, 1u) + 1u == gridDim.x) (void)atomicCAS(state, 0u, kCheckinGo);
    const uint64_t t0 = static_cast<uint64_t>(wall_clock64());
    uint32_t s;
    while ((s = atomic_load_u32(state)) == 0u) {
      if (static_cast<uint64_t>(wall_clock64()) - t0 >= ticks) {
        if (atomicCAS(state, 0u, kCheckinAbort) == 0u) atomicOr(err, kErrTailCheckin);
      } else {
        __builtin_amdgcn_s_sleep(1);
      }
    }
    *s_ok = s == kCheckinGo ? 1 : 0;
  }
  __syncthreads();
  return *s_ok != 0;
}

}  // namespace gcol
