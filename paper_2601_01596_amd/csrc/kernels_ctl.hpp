// The check that ends a round of the correction, shared by the control kernel and the plane pass.
#pragma once
#include "common.hpp"

namespace ffcz {

// What a control kernel tells the host after a check: one word per instance (or 1D signal) in
// pinned host memory, (call tag << 40) | (done << 32) | checks completed.  w null: nothing.
struct Post {
  unsigned long long* w;
  unsigned long long tag;
};
__device__ __forceinline__ void post_check(const Post& p, int64_t i, int checks, int done) {
  if (p.w)
    __hip_atomic_store(p.w + i, (p.tag << 40) | ((unsigned long long)done << 32) | (unsigned)checks, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Whether check k with vx violations ends the loop (Alg. 1: no coefficient violates; also at the
// round cap, or on non-finite input).
__device__ __forceinline__ bool check_stops(const DevState* st, int k, unsigned long long vx) {
  return st->nonfinite != 0 || (!st->fixed && vx == 0) || k >= st->max_iter;
}

// One lane: the outcome of check k of instance b into its state, the violation record and the
// posted word.  vz: clips of the pass that formed the checked iterate.
__device__ __forceinline__ void record_check(DevState* st, int k, unsigned long long vx, unsigned long long vz, bool stop,
                                             unsigned long long* viol, const Post& post, int64_t b) {
  viol[k] = vx;
  if (k == 0) st->v_first = vx;
  st->v_last = vx;
  if (k == 0) st->s_guard = vz;
  else st->s_clipped_total += vz;
  if (st->nonfinite) st->nonfinite_stop = 1;
  else if (stop) st->converged = vx == 0 ? 1 : 0;
  if (stop) st->done = 1;
  else st->round = k + 1;
  post_check(post, b, k + 1, stop);
}

}  // namespace ffcz
