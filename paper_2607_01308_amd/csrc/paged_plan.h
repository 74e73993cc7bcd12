// The guard of the paged table kernel: whether a plan is one of this set, and what
// is taken back when it is refused. Callable on the host too, so that a CPU test can
// run a workgroup's threads through it one after the other.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cmerge.h"

namespace cm {

// Thread tid of nt's part in refusing a plan: no Id and no task of the fused render
// (built for the plan before) is left, n_fresh holds `pages`, the plan `status`.
__host__ __device__ __forceinline__ void paged_refuse(int64_t* plan, int32_t n, int64_t pages,
                                                      int64_t status, int64_t* n_fresh,
                                                      int64_t* task_total, uint8_t* hsel, int tid,
                                                      int nt) {
  for (int i = tid; i < n; i += nt) hsel[i] = 1;
  if (tid == 0) {
    *n_fresh = pages;
    *task_total = 0;
    plan[CM_PLAN_STATUS] = status;
  }
}

// Called by every thread of the workgroup; sync is its barrier. False: nothing is to
// be done, the plan's status was an error already (n_fresh: 0) or it is now. Every
// thread has read the plan before the first one writes its status.
template <class Sync>
__host__ __device__ __forceinline__ bool paged_plan_usable(int64_t* plan, int32_t n, int b_shift,
                                                           int64_t nbo_cap, int64_t* n_fresh,
                                                           int64_t* task_total, uint8_t* hsel,
                                                           int tid, int nt, Sync sync) {
  const int64_t status = plan[CM_PLAN_STATUS];
  const int64_t n_u = plan[CM_PLAN_NUNIQUE];
  const int64_t T_out = plan[CM_PLAN_TOUT];
  sync();
  if (status != CM_OK) {
    if (tid == 0) *n_fresh = 0;
    return false;
  }
  const int64_t nbo = (T_out + ((int64_t)1 << b_shift) - 1) >> b_shift;
  if (n_u < 1 || n_u > n || nbo > nbo_cap) {     // not a plan of this set (checked on the
    paged_refuse(plan, n, 0, CM_ESHAPE, n_fresh, task_total, hsel, tid, nt);  // host for every
    return false;                                // other entry point)
  }
  return true;
}

}  // namespace cm
