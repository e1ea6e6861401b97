// Sessions: a traversal's levels run one after another inside one launch, each
// on as many workgroups as it can use.  This header holds what the traversals
// (session.hip: hops; wsssp.hip: weights) share: modes, records, barriers,
// queues.  A traversal is a policy class P:
//
//   P::Args                 kernel arguments
//   P::State                its words of the plan
//   P::begin(a, x, sh)      wave 0: plan of the first level; its one row to
//                             sh.stage[0] and the queue
//   P::step(a, x, sh, sink, c)        a grid or cluster level's work
//   P::solo(a, sh, cur, ncur, sink, c)  a solo level's work
//   P::scans(p)             the level sums c.scan
//   P::words(a)             64-node words of a scan level
//   P::kPiece               edges per queue entry
//   P::kAdmits              a level may have more members than the one before
//   P::join_ticks(p, words) how long the first level that needs others waits for them
//   P::advance(a, sh, nf, mf, scan, record)  wave 0, uniform arguments: the
//                             next level's plan from the sums over the
//                             workgroups (set_plan)
//   P::entry(key, deg, i), P::row_entry(key, deg)   queue entry of piece i of
//                             a row, of a whole row
//
// Modes.
//  * solo: at most kSoloCap frontier edges, workgroup 0 alone, frontier in LDS;
//  * cluster: at most kClusterEdges, the first 32 workgroups (one XCD's compute
//    units); each leaves its counters in a line of its own and reads everyone
//    else's, so a level ends one store-to-load hop after its slowest member,
//    with no atomic on the way;
//  * grid: K workgroups, K from the frontier's edges or, of a level over all
//    nodes, from their number, meeting at a counting barrier.
//
// Coherence.  Everything one level hands to the next (queue entries, bitmap
// words, counters, level records) is written with agent-scope stores or
// atomics, complete (s_waitcnt) before the workgroup reports the level's end,
// and read with agent-scope loads, which the reader's L1 does not serve.  So
// no cache is written back or invalidated between levels (an agent acquire
// fence in front of each level measured 15 us and more).
//
// Grid barrier.  32 consecutive ranks form a group with its own counter line
// (the memory side takes one atomic per line at a time, about 14 ns each: 256
// arrivals on one line measured 3.7 us, 32 measured 0.8).  An arrival is one
// non-returning add per counter, each carrying a count of arrivals in its top
// 16 bits; workgroup 0 polls the groups' lines until all have arrived, plans
// the next level from the sums it then holds and publishes its record: 64-bit
// words, each a 32-bit value with the record's number as its tag, so that a
// poll is one load per wave and needs no further read.
//
// Membership.  A barrier may only count workgroups that are running, and a
// plain launch promises nothing about that.  So each workgroup joins with an
// atomic when it starts; workgroup 0 gives ranks to those that have, when the
// first level that needs others comes up (after a wait of P::join_ticks), and to
// later ones ahead of each level: beside other work on the device few may start
// with the launch.  (Two callers on R-MAT 20, weighted: with the first list kept for
// the whole run one call in 20 took 50 ms instead of 2.)  A rank is kept for good,
// so that whoever is behind still belongs where it did.  Every wait is on workgroups
// that have joined, hence on running ones, and is bounded besides.  The bound is on
// a wait for the next record, so a long run of solo or cluster levels publishes one
// now and then.
#pragma once

#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"

namespace dawn {

constexpr int kSB = 512;              // threads per workgroup
constexpr int kSW = kSB / kWave;
constexpr int kStage = 2048;          // queue entries a workgroup stages in LDS (grid levels)
// Frontier edges (and rows) of a solo level: two a thread.  At 1,000 edges a
// solo level takes 4 to 5 us, as a cluster's does; at 400 it takes 3.
constexpr int kSoloCap = 1024;
// Push: frontier edges of a cluster level.  Around 30,000 edges cluster and
// grid levels both take 7 to 8 us.
constexpr int kClusterEdges = 32768;
// Scan levels (pull; weighted collections): 64-node words of a cluster level
// (four a wave).
constexpr int kClusterWords = 1024;
// Grid push: frontier edges per workgroup taking part (half a step of 64 a wave).
constexpr int kEdgesPerWg = 256;
// Solo or cluster levels between two records at most: some 15 ms, against the 10 s
// that workgroups without work wait for one.
constexpr unsigned kRecordLevels = 4096;

enum SessMode { kModeGrid = 1, kModeCluster = 2, kModeSolo = 3, kModeEnd = 4 };

// kNoRanks: no level has needed others yet.  kLaunchRanks: everyone had started when
// the first did.
enum SessRanks { kNoRanks = 0, kListed = 1, kLaunchRanks = 2 };

// The level to run: the policy's state, how it runs, and where its frontier's
// queue is.  32-bit words throughout, kept in LDS in the layout of the level
// record, so that publishing one is a read and a store per lane.
template <class State>
struct SessPlan {
  State u;
  unsigned step;                      // levels planned so far
  unsigned mode, K;
  unsigned fe;                        // out-edges of the frontier
  unsigned qp;                        // the queue's parity
  unsigned stride;                    // entries between its segments
  unsigned members;                   // workgroups with a rank (before any: of the launch)
  unsigned ranks;                     // where ranks stand (SessRanks)
  unsigned scan;                      // a level over all nodes, not over the queue
  unsigned seg_n[kSessSegs];          // entries of each segment
};
template <class P>
struct PlanWords {
  static constexpr int all = sizeof(SessPlan<typename P::State>) / 4;
  static constexpr int seg = all - kSessSegs;
  static_assert(all <= kSessRec && all <= kWave, "record words");
};

// The part of a workgroup's shared memory the queues use.
struct SessQueue {
  // grid: entries staged for the next frontier; solo: the two row lists
  u64 stage[kStage];
  int own[kSW][4 * kWave];            // per wave: which row an edge belongs to
  unsigned pre_g[kSessSegs + 1];      // first group of 64 entries of each segment
  unsigned rank;
  unsigned listed[kSessGroups];       // workgroup 0: those with a rank, as `joined`
  int all;                            // workgroup 0: every workgroup has joined, as far as
                                      //   it looked
  int go, ok;
  unsigned gb;                        // where the staged entries go in the sub-queue
  unsigned nf, mf, scan, n_out;       // this level's counters
};
static_assert(kStage >= 2 * kSoloCap, "solo lists alias the stage");

template <class P>
struct SessShared : SessQueue {
  SessPlan<typename P::State> p;
};

// Every earlier load, store and atomic of the wave is complete.
__device__ __forceinline__ void wait_all() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}
__device__ __forceinline__ void st_relaxed64(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// LDS written by some lanes of a wave is read by others: order the accesses.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// A value loaded only for its line: counts as used here.
__device__ __forceinline__ void keep(int x) { asm volatile("" ::"v"(x)); }
__device__ __forceinline__ unsigned uniform(unsigned x) {
  return (unsigned)__builtin_amdgcn_readfirstlane((int)x);
}

// How the planned level runs (wave 0).  end: there is none; scan: it goes over
// all nodes, `words` bitmap words of them; otherwise over a frontier with fe
// out-edges, solo up to solo_edges of them.
template <class P>
__device__ __forceinline__ void set_plan(SessShared<P>& sh, bool end, bool scan, u64 fe, int words,
                                         int solo_edges) {
  unsigned K = min(sh.p.members, (unsigned)kSessGroup), mode;
  if (end) {
    mode = kModeEnd;
  } else if (!scan && fe <= (u64)min(solo_edges, kSoloCap)) {
    mode = kModeSolo;
  } else if (K > 1 && (scan ? words <= kClusterWords : fe <= (u64)kClusterEdges)) {
    mode = kModeCluster;
  } else {
    const unsigned want = scan ? (unsigned)((words + kSW - 1) / kSW)
                               : (unsigned)((fe + kEdgesPerWg - 1) / kEdgesPerWg);
    mode = kModeGrid;
    K = min(sh.p.members, max(want, 1u));
  }
  if (lane_id() == 0) {
    sh.p.step += 1;
    sh.p.mode = mode;
    sh.p.K = K;
    sh.p.fe = (unsigned)fe;
    sh.p.scan = scan ? 1u : 0u;
  }
}

// How long a level waits for its members, where later levels may have more: at least
// kJoinTicks, and where there is much to do as long as a few would take for part of it
// (512 edges, or 64 nodes looked at, per 10 ns).
template <class State>
__device__ __forceinline__ unsigned long long admit_ticks(const SessPlan<State>& p, int words) {
  return kJoinTicks + (p.scan ? (unsigned)words : p.fe >> 9);
}

// Wave 0: segment sizes (lane s holds that of segment s) to LDS.
template <class P>
__device__ __forceinline__ void set_segments(SessShared<P>& sh, unsigned n) {
  const int lane = lane_id();
  const int incl = wave_incl_scan((int)((n + kWave - 1) / kWave));
  if (lane < kSessSegs) {
    sh.p.seg_n[lane] = n;
    sh.pre_g[lane + 1] = (unsigned)incl;
  }
  if (lane == 0) sh.pre_g[0] = 0;
}

// Wave 0 of workgroup 0 publishes record `gen` from LDS; everything its level
// reads is complete.  Then the counter slot of the record after it is zeroed
// (three in turn: its last use was two records ago): the stores complete
// before workgroup 0 arrives at this record's barrier, so before the next
// record can be.
template <class P>
__device__ __forceinline__ void sess_publish(SessCtrl* sc, SessShared<P>& sh, unsigned gen) {
  const int lane = lane_id();
  wave_sync();
  if (lane < PlanWords<P>::all)
    st_relaxed64(&sc->rec[lane],
                 ((u64)gen << 32) | reinterpret_cast<const unsigned*>(&sh.p)[lane]);
  SessSlot* z = &sc->slot[(gen + 1) % 3];
  if (lane < kSessGroups) {
    st_relaxed64(&z->grp[lane].w[0], 0ull);
    st_relaxed64(&z->grp[lane].w[1], 0ull);
    st_relaxed64(&z->grp[lane].w[2], 0ull);
  } else if (lane < kSessGroups + kSessStripes) {
    st_relaxed(&z->q[lane - kSessGroups].n, 0u);
  }
}

// Wave 0 waits for a record newer than `gen` and takes it over.  Returns its
// number, or 0 if the wait timed out.
template <class P>
__device__ __forceinline__ unsigned sess_poll(SessCtrl* sc, SessShared<P>& sh, unsigned gen,
                                              bool idle) {
  constexpr int kRWords = PlanWords<P>::all, kRSeg = PlanWords<P>::seg;
  const int lane = lane_id();
  const unsigned long long t0 = wall_clock64();
  for (;;) {
    const u64 w = lane < kRWords ? ld_relaxed(&sc->rec[lane]) : 0ull;
    const unsigned tag = (unsigned)(w >> 32);
    const unsigned first = uniform(tag);
    if (first > gen && __ballot(lane < kRWords && tag != first) == 0) {
      if (lane < kRSeg) reinterpret_cast<unsigned*>(&sh.p)[lane] = (unsigned)w;
      set_segments(sh, (unsigned)__shfl((int)(unsigned)w, lane < kSessSegs ? kRSeg + lane : 0, kWave));
      return first;
    }
    if (wall_clock64() - t0 > kBarrierTimeoutTicks) return 0;
    if (idle)
      __builtin_amdgcn_s_sleep(4);
    else
      __builtin_amdgcn_s_sleep(1);
  }
}

// Workgroups are numbered by layer, XCD and position there (consecutive ones go to
// the 8 XCDs in turn): word (layer, XCD), bit = position, so that 32 consecutive
// ranks share an XCD's L2.
__device__ __forceinline__ unsigned word_of(unsigned b) { return (b >> 8) * 8 + (b & 7); }
__device__ __forceinline__ unsigned bit_of(unsigned b) { return (b >> 3) & 31; }
__device__ __forceinline__ unsigned workgroup_of(unsigned word, unsigned bit) {
  return (word >> 3) * 256 + bit * 8 + (word & 7);
}

// Lane w: the workgroups of a launch of `grid` that have word w, as its bits.
__device__ __forceinline__ unsigned launch_word(int w, unsigned grid) {
  const int left = (int)grid - (w >> 3) * 256 - (w & 7);
  const int cnt = min((left + 7) >> 3, 32);
  return w >= kSessGroups || cnt <= 0 ? 0u : cnt == 32 ? ~0u : (1u << cnt) - 1u;
}

// Wave 0: workgroup b's rank if every workgroup has one.
__device__ __forceinline__ unsigned launch_rank(unsigned b) {
  const unsigned word = launch_word(lane_id(), gridDim.x);
  const int c = __popc(word);
  const unsigned before = (unsigned)__shfl(wave_incl_scan(c) - c, (int)word_of(b), kWave);
  return before + bit_of(b);
}

// Workgroup 0, wave 0 (lane w: word w): how many have joined.
__device__ __forceinline__ unsigned joined_count(SessCtrl* sc) {
  const unsigned w = lane_id() < kSessGroups ? (unsigned)ld_relaxed(&sc->joined[lane_id()].w) : 0u;
  return wave_sum((unsigned)__popc(w)) + 1;        // (itself does not)
}

// Workgroup 0, wave 0: ranks for those that have joined since.  True if any; they
// are in place then.
template <class P>
__device__ __forceinline__ bool sess_admit(SessCtrl* sc, SessShared<P>& sh) {
  const int lane = lane_id();
  const bool in = lane < kSessGroups;
  unsigned w = in ? (unsigned)ld_relaxed(&sc->joined[lane].w) : 0u;
  if (lane == 0) w |= 1u;
  const unsigned fresh = in ? w & ~sh.listed[lane] : 0u;
  const int c = __popc(fresh);
  const int incl = wave_incl_scan(c);
  const unsigned added = (unsigned)__builtin_amdgcn_readlane(incl, kWave - 1);
  if (!added) return false;
  const unsigned had = uniform(sh.p.ranks) == kNoRanks ? 0u : uniform(sh.p.members);
  unsigned r = had + (unsigned)(incl - c);
  for (unsigned f = fresh; f; f &= f - 1)
    st_relaxed(&sc->rank1[workgroup_of((unsigned)lane, (unsigned)__builtin_ctz(f))], ++r);
  if (in) sh.listed[lane] = w;
  if (lane == 0) {
    sh.p.members = had + added;
    sh.p.ranks = kListed;
    sh.all = had + added >= gridDim.x;
  }
  wait_all();
  wave_sync();
  return true;
}

struct SessCount {
  unsigned nf;      // nodes found (wave-uniform)
  unsigned mf;      // their out-edges (per lane)
  unsigned scan;    // scan levels: the policy's sum (per lane)
  int ahead;        // first target of a row found, loaded ahead of the next level
  int low;          // for the policy's use (per lane)
};

// Per-wave counters to the workgroup's.
__device__ __forceinline__ void add_counts(SessQueue& sh, const SessCount& c, bool scans) {
  const unsigned mf = wave_sum(c.mf);
  const unsigned sc = scans ? wave_sum(c.scan) : 0u;
  if (lane_id() == 0 && (c.nf | sc)) {
    atomicAdd(&sh.nf, c.nf);
    atomicAdd(&sh.mf, mf);
    if (sc) atomicAdd(&sh.scan, sc);
  }
}

// ------------------------------------------------- where found rows go --
// Each takes a whole wave's rows: a key (what the policy makes entries from)
// and the out-degree.

// Positions for `np` pieces per lane from an LDS counter; off: the lane's
// first, cnt: the wave's number (0: nothing to do).
struct Take {
  unsigned base, off, cnt;
};
__device__ __forceinline__ Take take(unsigned* counter, int np) {
  Take k{0, 0, 0};
  const u64 mask = __ballot(np > 0);
  if (!mask) return k;
  if (__ballot(np > 1) == 0) {
    k.off = (unsigned)__popcll(mask & lanes_below());
    k.cnt = (unsigned)__popcll(mask);
  } else {
    const int incl = wave_incl_scan(np);
    k.off = (unsigned)(incl - np);
    k.cnt = (unsigned)__builtin_amdgcn_readlane(incl, kWave - 1);
  }
  unsigned b = 0;
  if (lane_id() == 0) b = atomicAdd(counter, k.cnt);
  k.base = uniform(b);
  return k;
}

// Grid level: staged in LDS as pieces of at most P::kPiece edges; past the
// stage's end the wave reserves room in its workgroup's sub-queue itself.
// Cluster level (CLUSTER): straight to the workgroup's own segment, past its
// end to the clusters' common one.
template <class P, bool CLUSTER>
struct PieceSink {
  SessQueue& sh;
  u64* out;           // sub-queue, or own segment
  u64* rest;          // common segment
  int* own;           // this wave's marks
  unsigned* counter;  // entries of the sub-queue, or of the common segment
  unsigned cap;       // entries the stage, or the segment, holds

  __device__ __forceinline__ void add(bool found, int key, int deg) {
    const int np = found ? (deg + P::kPiece - 1) / P::kPiece : 0;
    const Take k = take(&sh.n_out, np);
    if (!k.cnt) return;
    const unsigned over = max(k.base, cap);
    unsigned gb = 0;
    if (k.base + k.cnt > cap) {
      if (lane_id() == 0) gb = atom_add(counter, k.base + k.cnt - over);
      gb = uniform(gb);
    }
    if (__ballot(np > 1) == 0) {
      if (np) store(k.base + k.off, over, gb, P::entry(key, deg, 0));
      return;
    }
    // rows of several pieces: 64 pieces of the wave's rows a round, whichever
    // rows they belong to (a loop over each lane's own pieces would last as
    // long as the longest row)
    const int lane = lane_id();
    for (int it = 0; it < (int)k.cnt; it += kWave) {
      const int at = (int)k.off - it;
      own[lane] = 0;
      wave_sync();
      if (np > 0 && at >= 0 && at < kWave) own[at] = lane;
      wave_sync();
      const int o = wave_incl_max(max(own[lane], 63 - __builtin_clzll(__ballot(np > 0 && at <= 0))));
      wave_sync();
      const int i = it + lane - __shfl((int)k.off, o, kWave);
      const u64 e = P::entry(__shfl(key, o, kWave), __shfl(deg, o, kWave), i);
      if (it + lane < (int)k.cnt) store(k.base + (unsigned)(it + lane), over, gb, e);
    }
  }
  __device__ __forceinline__ void store(unsigned pos, unsigned over, unsigned gb, u64 e) {
    if (pos >= cap)
      st_relaxed64(&(CLUSTER ? rest : out)[gb + (pos - over)], e);
    else if (CLUSTER)
      st_relaxed64(&out[pos], e);
    else
      sh.stage[pos] = e;
  }
};

// Solo level: whole rows to the other LDS list (a level finds no more nodes
// than it has edges, so they fit), and to segment 0 of the next queue in case
// the next level is not solo: stores nothing waits for here.
template <class P>
struct ListSink {
  SessQueue& sh;
  u64* list;
  u64* out;
  __device__ __forceinline__ void add(bool found, int key, int deg) {
    const bool ok = found && deg > 0;
    const Take k = take(&sh.n_out, ok ? 1 : 0);
    if (ok) {
      const u64 e = P::row_entry(key, deg);
      list[k.base + k.off] = e;
      st_relaxed64(&out[k.base + k.off], e);
    }
  }
};

// ---------------------------------------------- where a frontier's rows are --
constexpr u64 kNoEntry = ~0ull;   // a lane past the end
struct ListSrc {
  const u64* list;
  unsigned n;
  __device__ __forceinline__ u64 get(unsigned group, int lane) const {
    const unsigned i = group * kWave + (unsigned)lane;
    return i < n ? list[i] : kNoEntry;
  }
};

template <class P>
struct QueueSrc {
  const SessShared<P>& sh;
  const u64* q;
  unsigned pg;       // lane s: first group of segment s
  __device__ __forceinline__ u64 get(unsigned group, int lane) const {
    const int s = __popcll(__ballot(pg <= group)) - 1;
    const unsigned i = (group - (unsigned)__builtin_amdgcn_readlane((int)pg, s)) * kWave +
                       (unsigned)lane;
    return i < sh.p.seg_n[s] ? ld_relaxed(&q[(size_t)s * sh.p.stride + i]) : kNoEntry;
  }
};
template <class P>
__device__ __forceinline__ QueueSrc<P> queue_src(const SessShared<P>& sh, const u64* q) {
  const int lane = lane_id();
  return QueueSrc<P>{sh, q, lane < kSessSegs ? sh.pre_g[lane] : ~0u};
}

// The frontier's groups of 64 rows dealt over `nwaves` waves, this one being
// gw; with fewer groups than waves, a group's steps over several waves.  A
// wave walks the union of its group's rows in steps of E x 64 edges.  Which
// row an edge belongs to: each row marks the step's slot of its first edge in
// LDS, and a maximum scan carries the marks on (a few LDS accesses a step,
// where a binary search by lane permutes took 36 for 256 edges).
// row(entry, &rs, &deg): the lane's row; edges(owner, at, has): E edges per
// lane, of rows held by lanes owner[], at positions at[] past the lane-held
// `first` of that row (first = rs - exclusive prefix; given to edges()).
template <int E, class Src, class Row, class Edges>
__device__ __forceinline__ void walk_rows(int* own, unsigned ngroups, unsigned gw, unsigned nwaves,
                                          const Src& src, Row&& row, Edges&& edges) {
  const int lane = lane_id();
  // E = 1: a step each, if there are so many.  Longer steps: shares of two or
  // more a wave, so that unequal groups even out
  const unsigned split = max((E == 1 ? nwaves : 2 * nwaves + ngroups - 1) / max(ngroups, 1u), 1u);
  for (unsigned vw = gw; vw < ngroups * split; vw += nwaves) {
    const unsigned part = vw / ngroups;
    const u64 ent = src.get(vw - part * ngroups, lane);
    int rs = 0, deg = 0;
    row(ent, part, rs, deg);
    const int incl = wave_incl_scan(deg);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int excl = incl - deg;
    const int first = rs - excl;      // edge x of the union is entry first + x
    const int step = (int)split * E * kWave;
    int eb = (int)part * E * kWave;
    while (eb < total) {
#pragma unroll
      for (int q = 0; q < E; ++q) own[q * kWave + lane] = 0;
      wave_sync();
      if (deg > 0 && excl >= eb && excl < eb + E * kWave) own[excl - eb] = lane;
      wave_sync();
      // the row that covers the step's first edge
      int carry = 63 - __builtin_clzll(__ballot(deg > 0 && excl <= eb));
      int o[E], at[E];
      bool has[E];
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int x = eb + q * kWave + lane;
        o[q] = wave_incl_max(max(own[q * kWave + lane], carry));
        carry = __builtin_amdgcn_readlane(o[q], kWave - 1);
        at[q] = __shfl(first, o[q], kWave) + x;
        has[q] = x < total;
      }
      wave_sync();      // the marks are read before the next step clears them
      edges(o, at, has);
      // (eb + step may be past 2^31: a source's row is one entry, however long)
      if (total - eb <= step) break;
      eb += step;
    }
  }
}

// ---------------------------------------------------------------- grid level --
// Runs the level, then the barrier.  Returns the next record's number, or in
// workgroup 0 this one's if the next is still to be published (0: a wait timed out).
template <class P>
__device__ __forceinline__ unsigned grid_level(const typename P::Args& a, const SessArgs& x,
                                               SessShared<P>& sh, unsigned gen) {
  const int t = threadIdx.x, lane = lane_id();
  SessCtrl* sc = x.sc;
  SessSlot* slot = &sc->slot[gen % 3];
  const unsigned stripe = sh.rank % x.stripes;
  u64* qout = x.q[sh.p.qp ^ 1] + (size_t)stripe * x.qcap;
  unsigned* qn = &slot->q[stripe].n;
  const bool scans = P::scans(sh.p);
  {
    SessCount c{0, 0, 0, 0, 0};
    PieceSink<P, false> sink{sh, qout, qout, sh.own[t / kWave], qn, (unsigned)kStage};
    P::step(a, x, sh, sink, c);
    add_counts(sh, c, scans);
    keep(c.ahead);
  }
  wait_all();
  __syncthreads();
  const unsigned grp = sh.rank / kSessGroup;
  const unsigned n = min(sh.n_out, (unsigned)kStage);
  if (n) {
    if (t == 0) sh.gb = atom_add(qn, n);
    __syncthreads();
    for (unsigned i = (unsigned)t; i < n; i += kSB) st_relaxed64(&qout[sh.gb + i], sh.stage[i]);
    wait_all();
    __syncthreads();
  }
  if (t < kWave) {
    unsigned next = 0;
    if (lane < 3) {
      const unsigned v = lane == 0 ? sh.nf : lane == 1 ? sh.mf : sh.scan;
      atom_add(&slot->grp[grp].w[lane], (1ull << 48) | v);
    }
    wave_sync();
    if (lane == 0) sh.nf = sh.mf = sh.scan = sh.n_out = 0;
    if (sh.rank == 0) {
      const unsigned ngroups = (sh.p.K + kSessGroup - 1) / kSessGroup;
      const bool mem = lane < (int)ngroups;
      const unsigned long long t0 = wall_clock64();
      u64 w0 = 0, w1 = 0, w2 = 0;
      bool ok = true;
      for (;;) {
        if (mem) {
          w0 = ld_relaxed(&slot->grp[lane].w[0]);
          w1 = ld_relaxed(&slot->grp[lane].w[1]);
          w2 = ld_relaxed(&slot->grp[lane].w[2]);
        }
        const unsigned arrived = min(min((unsigned)(w0 >> 48), (unsigned)(w1 >> 48)),
                                     (unsigned)(w2 >> 48));
        const unsigned size = min((unsigned)kSessGroup, sh.p.K - (unsigned)lane * kSessGroup);
        if (!__ballot(mem && arrived < size)) break;
        if (wall_clock64() - t0 > kBarrierTimeoutTicks) {
          ok = false;
          break;
        }
      }
      if (ok) {
        const unsigned sq = lane < kSessStripes ? ld_relaxed(&slot->q[lane].n) : 0u;
        constexpr u64 low = (1ull << 48) - 1;
        const u64 nf = wave_sum(w0 & low), mf = wave_sum(w1 & low);
        const u64 sum = scans ? wave_sum(w2 & low) : 0ull;
        set_segments(sh, sq);
        P::advance(a, sh, (unsigned)nf, mf, sum, true);
        if (lane == 0) {
          sh.p.qp ^= 1;
          sh.p.stride = x.qcap;
        }
        next = gen;
        if (!P::kAdmits || uniform((unsigned)sh.all)) {
          sess_publish(sc, sh, gen + 1);
          next = gen + 1;
        }
      }
    } else {
      next = sess_poll(sc, sh, gen, false);
    }
    if (lane == 0) sh.ok = (int)next;
  }
  __syncthreads();
  return (unsigned)sh.ok;
}

// ------------------------------------------------------------- cluster levels --
// Cluster levels, one after another, by the first K (at most 32) workgroups.
// Every member reports each level in a line of its own (two lines, by level
// parity, tagged with the level's number) and reads all of them, so each holds the
// level's sums and takes the same decision.  A member cannot be two levels
// ahead of another, so two lines do.  On return sh holds the next level's
// plan, which only workgroup 0 uses; the others take it from the next record.
// After kRecordLevels levels all leave, whatever the next is.  Returns false if a
// wait timed out.
template <class P>
__device__ __forceinline__ bool cluster_run(const typename P::Args& a, const SessArgs& x,
                                            SessShared<P>& sh) {
  const int t = threadIdx.x, lane = lane_id();
  SessCtrl* sc = x.sc;
  const unsigned first = uniform(sh.p.step);
  for (;;) {
    const unsigned L = uniform(sh.p.step);
    const bool scans = P::scans(sh.p);
    // the counter of the next level was last read before this one began
    if (sh.rank == 0 && t == 0) st_relaxed(&sc->over[(L + 1) % 3].n, 0u);
    {
      SessCount c{0, 0, 0, 0, 0};
      u64* qout = x.q[sh.p.qp ^ 1];
      PieceSink<P, true> sink{sh, qout + (size_t)sh.rank * x.ccap,
                           qout + (size_t)kSessGroup * x.ccap, sh.own[t / kWave],
                               &sc->over[L % 3].n, x.ccap};
      P::step(a, x, sh, sink, c);
      add_counts(sh, c, scans);
      keep(c.ahead);
    }
    wait_all();
    __syncthreads();
    if (t < kWave) {
      const unsigned n = sh.n_out;
      const unsigned mine = lane == 0 ? n : lane == 1 ? sh.nf : lane == 2 ? sh.mf : sh.scan;
      if (lane < 4)
        st_relaxed64(&sc->crec[L & 1][sh.rank].w[lane], ((u64)L << 32) | mine);
      const bool mem = lane < (int)sh.p.K;
      const u64* line = sc->crec[L & 1][lane & (kSessGroup - 1)].w;
      const unsigned long long t0 = wall_clock64();
      u64 w0 = 0, w1 = 0, w2 = 0, w3 = 0;
      int state = 0;      // 1: complete, 2: a later cluster run has begun
      for (;;) {
        if (mem) {
          w0 = ld_relaxed(line);
          w1 = ld_relaxed(line + 1);
          w2 = ld_relaxed(line + 2);
          w3 = ld_relaxed(line + 3);
        }
        const unsigned lo = min(min((unsigned)(w0 >> 32), (unsigned)(w1 >> 32)),
                                min((unsigned)(w2 >> 32), (unsigned)(w3 >> 32)));
        const unsigned hi = max(max((unsigned)(w0 >> 32), (unsigned)(w1 >> 32)),
                                max((unsigned)(w2 >> 32), (unsigned)(w3 >> 32)));
        if (__ballot(mem && hi > L)) state = 2;
        else if (!__ballot(mem && lo != L)) state = 1;
        if (state) break;
        if (wall_clock64() - t0 > kBarrierTimeoutTicks) break;
      }
      if (state == 1) {
        const unsigned cnt = mem ? (unsigned)w0 : 0u;
        const u64 nf = wave_sum(mem ? (unsigned)w1 : 0u);
        const u64 mf = wave_sum(mem ? (unsigned)w2 : 0u);
        const u64 sum = scans ? (u64)wave_sum(mem ? (unsigned)w3 : 0u) : 0ull;
        unsigned seg = min(cnt, x.ccap);
        if (__ballot(cnt > x.ccap)) {
          const unsigned ov = ld_relaxed(&sc->over[L % 3].n);
          if (lane == kSessGroup) seg = ov;
        }
        set_segments(sh, seg);
        P::advance(a, sh, (unsigned)nf, mf, sum, sh.rank == 0);
        if (lane == 0) {
          sh.p.qp ^= 1;
          sh.p.stride = x.ccap;
        }
      }
      // (state 2 too: the counters are the reported level's, and the workgroup goes on
      // to a level of the later run)
      if (lane == 0) {
        sh.nf = sh.mf = sh.scan = sh.n_out = 0;
        sh.ok = state;
      }
    }
    __syncthreads();
    if (sh.ok != 1) return sh.ok == 2;
    if (sh.p.mode != kModeCluster || L - first >= kRecordLevels - 1) {
      // clear for the next run, which starts with a record of workgroup 0
      // after its next wait for its stores
      if (sh.rank == 0 && t < 3) st_relaxed(&sc->over[t].n, 0u);
      return true;
    }
  }
}

// ---------------------------------------------------------------- solo levels --
// Workgroup 0 alone, up to kRecordLevels levels.  On entry `cur` holds ncur rows and
// sh.p the level to run; on return sh.p is the next level, its queue written, or the
// end.
template <class P>
__device__ __forceinline__ void solo_run(const typename P::Args& a, const SessArgs& x,
                                         SessShared<P>& sh, u64* cur, unsigned ncur) {
  const int t = threadIdx.x, wv = t / kWave, lane = lane_id();
  int ahead = 0;
  for (unsigned ran = 1;; ++ran) {
    u64* nxt = cur == sh.stage ? sh.stage + kSoloCap : sh.stage;
    {
      SessCount c{0, 0, 0, 0, 0};
      ListSink<P> sink{sh, nxt, x.q[sh.p.qp ^ 1]};
      P::solo(a, sh, cur, ncur, sink, c);
      add_counts(sh, c, false);
      keep(ahead);        // (of the level before)
      ahead = c.ahead;
      if (wv == kSW - 1 && !sh.all) {
        // the wave that is first out of work looks who has joined
        if (sh.p.ranks == kNoRanks && joined_count(x.sc) >= gridDim.x && lane == 0) sh.all = 1;
      }
    }
    __syncthreads();
    ncur = uniform(sh.n_out);
    cur = nxt;
    if (t < kWave) {
      const unsigned nf = uniform(sh.nf), mf = uniform(sh.mf);
      P::advance(a, sh, nf, mf, 0ull, true);
      wave_sync();
      const bool solo = sh.p.mode == kModeSolo && ran < kRecordLevels;
      if (!solo) set_segments(sh, lane == 0 ? ncur : 0u);
      if (lane == 0) {
        sh.nf = sh.mf = 0;
        sh.go = solo ? 1 : 0;
        if (!solo) {
          sh.p.qp ^= 1;
          sh.p.stride = x.qcap;
        }
      }
    }
    __syncthreads();
    if (t == 0) sh.n_out = 0;
    // this level's queue entries are complete before the next level's (the
    // same places), or before the next record
    wait_all();
    __syncthreads();
    if (!sh.go) break;
  }
  keep(ahead);
}

// The kernel body: kSB threads per workgroup, gridDim.x at most kSessGroups x
// kSessGroup.
template <class P>
__device__ __forceinline__ void session(const typename P::Args& a, const SessArgs& x,
                                        SessShared<P>& sh) {
  const unsigned long long t_start = wall_clock64();
  const int t = threadIdx.x, lane = lane_id();
  const unsigned bid = blockIdx.x;
  SessCtrl* sc = x.sc;
  if (t == 0) {
    sh.nf = sh.mf = sh.scan = sh.n_out = 0;
    sh.ok = 1;
    sh.all = 0;
    if (bid != 0) atom_or(&sc->joined[word_of(bid)].w, 1ull << bit_of(bid));
  }
  if (t < kSessGroups) sh.listed[t] = 0;
  if (t < kWave) {
    const unsigned r = launch_rank(bid);
    if (lane == 0) sh.rank = r;
  }
  __syncthreads();
  unsigned gen = 0;
  bool ranked = bid == 0, lead = false;    // lead: workgroup 0 holds the next plan
  if (bid == 0) {
    if (t < kWave) {
      if (lane == 0) {
        sh.p.step = 0;
        sh.p.mode = 0;
        sh.p.qp = 0;
        sh.p.stride = x.qcap;
        sh.p.members = gridDim.x;
        sh.p.ranks = kNoRanks;
      }
      wave_sync();
      P::begin(a, x, sh);
      set_segments(sh, lane == 0 ? 1u : 0u);
      wait_all();
    }
    __syncthreads();
    if (sh.p.mode == kModeSolo) solo_run(a, x, sh, sh.stage, 1);
    lead = true;
  } else {
    if (t < kWave) {
      const unsigned g = sess_poll(sc, sh, 0, false);
      if (lane == 0) sh.ok = (int)g;
    }
    __syncthreads();
    gen = (unsigned)sh.ok;
    if (!gen) return;
  }
  for (;;) {
    if (lead) {
      if (t < kWave) {
        const unsigned mode = uniform(sh.p.mode);
        const bool wide = mode == kModeGrid || mode == kModeCluster;
        const bool first = wide && uniform(sh.p.ranks) == kNoRanks;
        bool all = uniform((unsigned)sh.all) != 0;
        if (first) {
          // the first level that needs others
          const unsigned long long ticks = P::join_ticks(sh.p, P::words(a));
          while (!all && wall_clock64() - t_start <= ticks) all = joined_count(sc) >= gridDim.x;
          if (all && lane == 0) sh.p.ranks = kLaunchRanks, sh.all = 1;
        }
        // (if more get in, the plan was made for other members)
        if (wide && !all && (first || P::kAdmits) && sess_admit(sc, sh))
          set_plan<P>(sh, false, sh.p.scan != 0, uniform(sh.p.fe), P::words(a), 0);
        sess_publish(sc, sh, gen + 1);
      }
      gen += 1;
      lead = false;
      __syncthreads();
    }
    if (sh.p.mode == kModeEnd) return;
    if (!ranked && sh.p.ranks != kNoRanks) {
      if (sh.p.ranks == kListed) {
        __syncthreads();
        if (t == 0) sh.rank = ld_relaxed(&sc->rank1[bid]) - 1u;     // (none: the largest)
        __syncthreads();
      }
      ranked = sh.rank != ~0u;
      if (!ranked && !P::kAdmits) return;
    }
    // (a rank given since the record is past its members)
    const bool mine = sh.p.mode == kModeSolo ? bid == 0 : ranked && sh.rank < sh.p.K;
    bool poll = !mine;
    if (mine && sh.p.mode == kModeGrid) {
      const unsigned next = grid_level(a, x, sh, gen);
      if (!next) return;
      lead = next == gen;
      gen = next;
    } else if (mine) {
      if (sh.p.mode == kModeCluster) {
        if (!cluster_run(a, x, sh)) return;
        poll = bid != 0;
        lead = bid == 0;
      }
      if (bid == 0 && sh.p.mode == kModeSolo) {
        // the frontier from the queue: at most kSoloCap rows
        __syncthreads();
        const QueueSrc<P> src = queue_src(sh, x.q[sh.p.qp]);
        for (unsigned g = (unsigned)(t / kWave); g < sh.pre_g[kSessSegs]; g += kSW) {
          const u64 e = src.get(g, lane);
          const Take k = take(&sh.n_out, e != kNoEntry ? 1 : 0);
          if (e != kNoEntry && k.base + k.off < (unsigned)kSoloCap) sh.stage[k.base + k.off] = e;
        }
        __syncthreads();
        const unsigned ncur = min(sh.n_out, (unsigned)kSoloCap);
        __syncthreads();
        if (t == 0) sh.n_out = 0;
        __syncthreads();
        solo_run(a, x, sh, sh.stage, ncur);
        lead = true;
      }
    }
    if (poll) {
      __syncthreads();
      if (t < kWave) {
        const unsigned g = sess_poll(sc, sh, gen, !mine);
        if (lane == 0) sh.ok = (int)g;
      }
      __syncthreads();
      gen = (unsigned)sh.ok;
      if (!gen) return;
    }
  }
}

// Workgroups of a session's launch: per_cu per compute unit, divided by `share`, but no
// more than a level can use (words: 64-node words of a scan level; m: edges).  A
// session holds what it has to its end, so calls that share the device (ctx_share)
// take a part each: sessions that take all of it run one after another, and whoever
// comes next starts with what the last one left.
// Calls a second by one, two and four callers, with all of it to each and now: R-MAT 20
// 10,900, 7,800, 7,400 and 10,800, 14,500, 14,700 (a launch per level: 5,300, 6,000,
// 5,700); R-MAT 17 beside a caller on a long grid 320 and 17,000 (3,800).
inline int sess_grid(const Ctx* ctx, int per_cu, int share, int words, long long m) {
  const long long useful = std::max<long long>((words + kSW - 1) / kSW,
                                               (m + kEdgesPerWg - 1) / kEdgesPerWg);
  return (int)std::max<long long>(
      1, std::min<long long>({useful, (long long)std::max(per_cu * ctx->num_cu / share, kSessGroup),
                              (long long)kSessGroups * kSessGroup}));
}

}  // namespace dawn
