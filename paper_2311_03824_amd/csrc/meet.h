// Workgroups of one launch that share the phases of a computation and meet at a counter
// between them, with any number of them resident.
//
// A launch cannot know how many of its workgroups the device will hold at once: other streams,
// other processes, a CU mask or a partition may leave room for a few only, and a workgroup that
// waits keeps its place.  So the workgroups first take a roll call.  Each arrival counts itself;
// when the last one has come, or when one has waited kRollGrace for the rest, the roll is closed,
// and the work of every phase is dealt to the workgroups on it.  One that comes later ends at
// once.  From then on a wait is only ever for workgroups that are running, so every wait
// ends.  The work is dealt in units whose results do not depend on who computes them, so neither do
// the results on the roll.
#pragma once
#include "common.h"

namespace altg {

constexpr int kRollClosed = 1 << 30;
// 2 ms in ticks of the 100 MHz wall clock: longer than the kernels whose workgroups give way to
// these within one launch of theirs, shorter than what a start with a partial roll takes.
constexpr int kRollGrace = 200000;

struct Meeting {
  Ctl* ctl;                // bar, roll and members are zero at launch (launch_reset_ctl)
  int id = 0, count = 1;   // this workgroup's number on the roll, the workgroups on it
  unsigned target = 0;
  __device__ explicit Meeting(Ctl* c) : ctl(c) {}

  // False: this workgroup came after the roll was closed and ends.  grace in wall clock ticks; sh: LDS.
  __device__ __forceinline__ bool join(int grace, int2* sh) {
    if (gridDim.x == 1) return true;
    if (threadIdx.x == 0) {
      const int mine = __hip_atomic_fetch_add(&ctl->roll, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int c = 0;
      if (!(mine & kRollClosed)) {
        if (mine == (int)gridDim.x - 1)
          __hip_atomic_store(&ctl->members, (int)gridDim.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long t0 = wall_clock64();
        while ((c = __hip_atomic_load(&ctl->members, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
          if (wall_clock64() - t0 >= grace) {
            const int n = __hip_atomic_fetch_or(&ctl->roll, kRollClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!(n & kRollClosed))   // the one that closes it writes the count (at least itself)
              __hip_atomic_store(&ctl->members, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      *sh = make_int2(mine, c);
    }
    __syncthreads();
    const int2 v = *sh;
    __syncthreads();
    id = v.x;
    count = v.y;
    return v.y != 0;
  }

  // Every workgroup's earlier writes are visible to all of them after it.  A wave waits for its
  // own stores first: the barrier does not, and the release by thread 0 waits for wave 0's alone.
  __device__ __forceinline__ void operator()() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (count == 1) return;
    target += count;
    if (threadIdx.x == 0) {
      __hip_atomic_fetch_add(&ctl->bar, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      while ((int)((unsigned)__hip_atomic_load(&ctl->bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0)
        __builtin_amdgcn_s_sleep(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
  }
};

}  // namespace altg
