// Device code shared by the single-source kernels (sssp.hip, session.hip).
#pragma once

#include "device_util.hpp"
#include "internal.hpp"

namespace dawn {

struct SlotSum {
  unsigned nf;
  u64 mf;
  u64 edges;
};

// Fold level st.level's counters into the state and choose level st.level+1.
// Direction switch in the style of direction-optimising BFS: go bottom-up
// (pull) when the frontier's out-edges exceed the unvisited out-edges / alpha
// while the frontier grows, and back top-down (push) when the frontier falls
// under n / beta while it shrinks.
__device__ __forceinline__ void decide(const SsspArgs& a, LevelState& st, const SlotSum& sl, bool record) {
  const int L = st.level;
  if (sl.nf > 0) st.last_nonempty = L;
  st.mu -= (long long)sl.mf;
  st.edges_total += sl.edges;
  st.source_edges += sl.mf;
  st.reached += sl.nf;
  if (record && L < a.lrec) a.level_nf[L] = (int32_t)sl.nf;
  const unsigned prev = st.prev_nf;
  st.prev_nf = sl.nf;
  if (sl.mf == 0) {
    st.done = 1;
    return;
  }
  if (L + 1 > a.n) {
    st.done = 2;
    return;
  }
  bool pull = st.pull;
  if (a.mode == 1) {
    pull = false;
  } else if (a.mode == 2) {
    pull = true;
  } else if (!pull) {
    if ((double)sl.mf * (double)a.alpha > (double)st.mu && sl.nf > prev) pull = true;
  } else {
    if ((double)sl.nf * (double)a.beta < (double)a.n && sl.nf < prev) pull = false;
  }
  st.pull = pull ? 1 : 0;
  st.level = L + 1;
  if (pull) st.pull_levels++; else st.push_levels++;
  if (record && st.level < a.lrec) a.level_dir[st.level] = pull ? 2 : 1;
}

// The state a launch of parity `parity` leaves, to the host mirror (one
// thread).  `ended`: this launch found the end of the traversal, so the end
// stamp and tag follow, the tag ordered after the rest by a system-scope
// release, which also writes back this XCD's L2: the host returns on the tag
// and its caller may read the distances at once.  Distances stored by other
// waves of the workgroup must be complete before (their waves wait for
// their stores ahead of the barrier that precedes the report); those of
// earlier launches were written back when those launches ended.
__device__ __forceinline__ void report(const SsspArgs& a, int parity, const LevelState& s,
                                       bool ended) {
  if (!a.hm) return;
  a.hm->st[parity] = s;
  if (ended) {
    a.hm->t_end = wall_clock64();
    __hip_atomic_store(&a.hm->end_tag, (a.seq << 1) | (unsigned)parity, __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace dawn
