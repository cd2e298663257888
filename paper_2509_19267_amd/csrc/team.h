// The workgroups of a launch that are on the device together (gridcg.hip,
// pcg.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace rg {

// Nothing says that all workgroups of a launch run at the same time: another
// stream's launch may hold the other half of the compute units, and wait as
// well.  So every workgroup counts itself in; the first one waits a moment
// (TEAM_WAIT of the 100 MHz clock) for the others and fixes the number; who
// comes later leaves.  The shares of those are taken by the ones that are
// there.  Counts go on over a solve's launches: each adds the whole grid.
// Ctrl::team_max (0: none) caps the number, so that a test can have every
// size of team: the workgroups above it leave as late ones do.  A kernel that
// needs at least `least` of them waits for those (bounded, Ctrl::sync_fail).
constexpr long long TEAM_WAIT = 20000;   // 200 us
struct Team {
  int rank, size;

  // s_old: workgroups counted in before this one (thread 0's)
  __device__ __forceinline__ void enter(unsigned long long *tm,
                                        unsigned long long *s_old) {
    if (threadIdx.x == 0)
      *s_old = __hip_atomic_fetch_add(&tm[0], 1ull, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
  }
  // false for a workgroup that came too late
  __device__ __forceinline__ bool settle(unsigned long long *tm,
                                         const unsigned long long *s_old,
                                         Ctrl *ctrl, int least = 1) {
    __shared__ int s_rank, s_size;
    if (threadIdx.x == 0) {
      const unsigned long long V = gridDim.x, old = *s_old;
      const unsigned long long launch = old / V;
      const unsigned long long tag = launch + 1;
      unsigned long long n = 0;
      s_rank = (int)(old % V);
      if (old % V == 0) {
        const unsigned long long cap = (unsigned long long)ctrl->team_max;
        unsigned long long want = cap > 0 && cap < V ? cap : V;
        if (want < (unsigned long long)least) want = least;
        const long long t0 = wall_clock64();
        int64_t spins = 0;
        do n = ld_agent(&tm[0]) - launch * V;
        while (n < want && (wall_clock64() - t0 < TEAM_WAIT ||
                            (n < (unsigned long long)least &&
                             ++spins <= GRID_SPIN_MAX)));
        if (n > want) n = want;
        if (n < (unsigned long long)least) {
          st_agent(&ctrl->sync_fail, 1);
          n = 0;
        }
        st_agent(&tm[1], tag << 16 | n);
      } else {
        int64_t spins = 0;
        while (((n = ld_agent(&tm[1])) >> 16) != tag) {
          if (++spins > GRID_SPIN_MAX) {
            st_agent(&ctrl->sync_fail, 1);
            n = 0;
            break;
          }
        }
        n &= 0xffff;
      }
      s_size = (int)n;
    }
    __syncthreads();
    rank = __builtin_amdgcn_readfirstlane(s_rank);
    size = __builtin_amdgcn_readfirstlane(s_size);
    return rank < size;
  }
};

}  // namespace rg
