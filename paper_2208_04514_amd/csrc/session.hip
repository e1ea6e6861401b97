// Single-source traversal in one launch: levels run one after another inside
// the kernel, each on as many workgroups as it can use.
//
// The level step is the one of sssp.hip (push: Section 3.3, Algorithm 2; pull:
// Section 3.2, Algorithm 1 with the early exit).  What differs is where a level
// ends.  A launch per level costs about 10 us even when the level has a few
// hundred edges (dispatch, first reads of a state the other XCDs wrote, the
// write-back at the end), and most levels of a road-like graph, and the first
// and last of any graph, are that small.  Here a level runs in one of
//
//  * solo: at most kSoloCap frontier edges, workgroup 0 alone, frontier in LDS;
//  * cluster: at most kClusterEdges, the first 32 workgroups (one XCD's compute
//    units); each leaves its counters in a line of its own and reads everyone
//    else's, so a level ends one store-to-load hop after its slowest member,
//    with no atomic on the way;
//  * grid: K workgroups, K from the frontier's edges (push) or the bitmap's
//    words (pull), meeting at a counting barrier.
//
// Coherence.  Everything one level hands to the next (queue entries, bitmap
// words, counters, level records) is written with agent-scope stores or
// atomics, complete (s_waitcnt) before the workgroup reports the level's end,
// and read with agent-scope loads, which the reader's L1 does not serve.  So
// no cache is written back or invalidated between levels (an agent acquire
// fence in front of each level measured 15 us and more).  Distances are plain
// stores nothing reads before the launch has ended.
//
// Grid barrier.  32 consecutive ranks form a group with its own counter line
// (the memory side takes one atomic per line at a time, about 14 ns each: 256
// arrivals on one line measured 3.7 us, 32 measured 0.8).  The last arrival of
// the last group sums the counters, applies the direction rule and publishes
// the next level's record: 64-bit words, each a 32-bit value with the record's
// number as its tag, so that a poll is one load per wave and needs no further
// read.
//
// Bound: a level's chain of dependent memory round trips (queue entry, targets,
// claim with the row bounds, queue store, report), about 2 us solo, 4.5 in a
// cluster, 7 in the grid, until a level has some 10^5 edges; from there the
// claims and bitmap reads.  Per source against a launch per level (MI355X):
// R-MAT 20 186 -> 95 us; grid 2048^2 (some 130 levels) 2.64 -> 1.41 ms; grid
// 1023 x 1025 without shortcuts (some 1,500 levels) 17.3 -> 6.5 ms; uniform
// n = 4096 70 -> 51 us.
//
// Membership.  A barrier may only count workgroups that are running, and a
// plain launch promises nothing about that.  So each workgroup joins with an
// atomic when it starts; workgroup 0 closes the list when the first level
// that needs others comes up; whoever starts later leaves at once.  Every
// wait is on workgroups that have joined, hence on running ones, and is
// bounded besides.
#include <string.h>

#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"
#include "sssp_dev.hpp"

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
// Pull: bitmap words of a cluster level (four a wave).
constexpr int kClusterWords = 1024;
// Grid push: frontier edges per workgroup taking part (half a step of 64 a wave).
constexpr int kEdgesPerWg = 256;
constexpr u64 kClosed = 1ull << 63;

enum SessMode { kModeGrid = 1, kModeCluster = 2, kModeSolo = 3, kModeEnd = 4 };

// The level to run: its state (LevelState's fields), how it runs, and where its
// frontier's queue is.  32-bit words throughout, kept in LDS in the layout of
// the level record, so that publishing one is a read and a store per lane.
struct SessPlan {
  unsigned level, cur, pull, done;
  unsigned mu, last_nonempty, push_levels, pull_levels, prev_nf;
  unsigned edges_lo, edges_hi, source_edges, reached;
  unsigned mode, K;
  unsigned fe;                        // out-edges of the frontier
  unsigned qp;                        // the queue's parity
  unsigned stride;                    // entries between its segments
  unsigned full;                      // every workgroup of the launch has joined
  unsigned seg_n[kSessSegs];          // entries of each segment
};
constexpr int kRWords = sizeof(SessPlan) / 4;
constexpr int kRSeg = kRWords - kSessSegs;
static_assert(kRWords <= kSessRec && kRWords <= kWave, "record words");

struct SessShared {
  // grid: entries staged for the next frontier; solo: the two row lists
  u64 stage[kStage];
  int own[kSW][4 * kWave];            // per wave: which row an edge belongs to
  SessPlan p;
  unsigned pre_g[kSessSegs + 1];      // first group of 64 entries of each segment
  unsigned rank, members;
  int go, ok;
  unsigned gb;                        // where the staged entries go in the sub-queue
  unsigned nf, mf, edges, n_out;      // this level's counters
};
static_assert(kStage >= 2 * kSoloCap, "solo lists alias the stage");

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
__device__ __forceinline__ u64 entry_of(int rs, int deg) {
  return (u64)(unsigned)rs | ((u64)(unsigned)deg << 32);
}
__device__ __forceinline__ unsigned uniform(unsigned x) {
  return (unsigned)__builtin_amdgcn_readfirstlane((int)x);
}

__device__ __forceinline__ LevelState sess_state(const SessPlan& p) {
  LevelState st;
  st.level = (int)p.level;
  st.cur = (int)p.cur;
  st.pull = (int)p.pull;
  st.done = (int)p.done;
  st.mu = (long long)p.mu;
  st.last_nonempty = (int)p.last_nonempty;
  st.push_levels = (int)p.push_levels;
  st.pull_levels = (int)p.pull_levels;
  st.launches = 1;
  st.prev_nf = p.prev_nf;
  st.mbar = 0;
  st.edges_total = (u64)p.edges_lo | ((u64)p.edges_hi << 32);
  st.source_edges = p.source_edges;
  st.reached = p.reached;
  return st;
}

// Fold the counters of the level run into its state and choose the next level.
// Whole wave, uniform arguments: every lane computes the same.  A pull level
// has made the other bitmap the current one.
__device__ __forceinline__ LevelState sess_decide(const SsspArgs& a, const SessPlan& p,
                                                  const SlotSum& sum, bool record) {
  LevelState st = sess_state(p);
  st.done = 0;
  st.cur ^= st.pull;
  decide(a, st, sum, record && lane_id() == 0);
  return st;
}

// A push level whose frontier (fe out-edges) workgroup 0 runs alone.
__device__ __forceinline__ bool is_solo(const SsspArgs& a, const LevelState& st, u64 fe) {
  return !st.done && !st.pull && fe <= (u64)min(a.small_edges, kSoloCap);
}

// The level decided in st, and how it runs (fe: the frontier's out-edges).
__device__ __forceinline__ void sess_plan(const SsspArgs& a, SessPlan& p, const LevelState& st,
                                          u64 fe, unsigned members) {
  unsigned K = min(members, (unsigned)kSessGroup), mode;
  if (st.done) {
    mode = kModeEnd;
  } else if (is_solo(a, st, fe)) {
    mode = kModeSolo;
  } else if (K > 1 && (st.pull ? a.nw <= kClusterWords : fe <= (u64)kClusterEdges)) {
    mode = kModeCluster;
  } else {
    const unsigned want = st.pull ? (unsigned)((a.nw + kSW - 1) / kSW)
                                  : (unsigned)((fe + kEdgesPerWg - 1) / kEdgesPerWg);
    mode = kModeGrid;
    K = min(members, max(want, 1u));
  }
  if (lane_id() == 0) {
    p.level = (unsigned)st.level;
    p.cur = (unsigned)st.cur;
    p.pull = (unsigned)st.pull;
    p.done = (unsigned)st.done;
    p.mu = (unsigned)st.mu;
    p.last_nonempty = (unsigned)st.last_nonempty;
    p.push_levels = (unsigned)st.push_levels;
    p.pull_levels = (unsigned)st.pull_levels;
    p.prev_nf = st.prev_nf;
    p.edges_lo = (unsigned)st.edges_total;
    p.edges_hi = (unsigned)(st.edges_total >> 32);
    p.source_edges = (unsigned)st.source_edges;
    p.reached = (unsigned)st.reached;
    p.mode = mode;
    p.K = K;
    p.fe = (unsigned)fe;
    if (mode == kModeEnd) a.ctrl->st[1] = st;
  }
}

// Wave 0: segment sizes (lane s holds that of segment s) to LDS.
__device__ __forceinline__ void set_segments(SessShared& sh, unsigned n) {
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
__device__ __forceinline__ void sess_publish(SessCtrl* sc, SessShared& sh, unsigned gen) {
  const int lane = lane_id();
  wave_sync();
  if (lane < kRWords)
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
__device__ __forceinline__ unsigned sess_poll(SessCtrl* sc, SessShared& sh, unsigned gen,
                                              bool idle) {
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

// Wave 0: rank and member count from the closed list (lane w holds word w).
__device__ __forceinline__ void sess_rank(const unsigned word, SessShared& sh, unsigned wi,
                                          unsigned bi) {
  const int c = __popc(word);
  const int incl = wave_incl_scan(c);
  const unsigned mine = (unsigned)__shfl((int)word, (int)wi, kWave);
  const unsigned before = (unsigned)__shfl(incl - c, (int)wi, kWave);
  const unsigned all = (unsigned)__builtin_amdgcn_readlane(incl, kWave - 1);
  if (lane_id() == 0) {
    sh.rank = before + (unsigned)__popc(mine & ((1u << bi) - 1u));
    sh.members = all;
  }
}

// Lane w: the workgroups of a launch of `grid` that have word w, as its bits.
__device__ __forceinline__ unsigned launch_word(int w, unsigned grid) {
  const int left = (int)grid - (w >> 3) * 256 - (w & 7);
  const int cnt = min((left + 7) >> 3, 32);
  return w >= kSessGroups || cnt <= 0 ? 0u : cnt == 32 ? ~0u : (1u << cnt) - 1u;
}

struct SessCount {
  unsigned nf;      // wave-uniform
  unsigned mf;      // per lane
  unsigned edges;   // per lane (pull)
  int ahead;        // first target of a row found, loaded ahead of the next level
};

// ------------------------------------------------- where found rows go --
// Each takes a whole wave's found nodes (row start, out-degree).

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

// Grid level: staged in LDS as pieces of at most kPiece edges; past the
// stage's end the wave reserves room in its workgroup's sub-queue itself.
// Cluster level (CLUSTER): straight to the workgroup's own segment, past its
// end to the clusters' common one.
template <bool CLUSTER>
struct PieceSink {
  SessShared& sh;
  u64* out;           // sub-queue, or own segment
  u64* rest;          // common segment
  unsigned* counter;  // entries of the sub-queue, or of the common segment
  unsigned cap;       // entries the stage, or the segment, holds

  __device__ __forceinline__ void add(bool found, int rs, int deg) {
    const int np = found ? (deg + kPiece - 1) / kPiece : 0;
    const Take k = take(&sh.n_out, np);
    if (!k.cnt) return;
    const unsigned over = max(k.base, cap);
    unsigned gb = 0;
    if (k.base + k.cnt > cap) {
      if (lane_id() == 0) gb = atom_add(counter, k.base + k.cnt - over);
      gb = uniform(gb);
    }
    for (int i = 0; i < np; ++i) {
      const unsigned pos = k.base + k.off + (unsigned)i;
      const u64 e = entry_of(rs + i * kPiece, min(kPiece, deg - i * kPiece));
      if (pos >= cap)
        st_relaxed64(&(CLUSTER ? rest : out)[gb + (pos - over)], e);
      else if (CLUSTER)
        st_relaxed64(&out[pos], e);
      else
        sh.stage[pos] = e;
    }
  }
};

// Solo level: whole rows to the other LDS list (a level finds no more nodes
// than it has edges, so they fit), and to segment 0 of the next queue in case
// the next level is not solo: stores nothing waits for here.
struct ListSink {
  SessShared& sh;
  u64* list;
  u64* out;
  __device__ __forceinline__ void add(bool found, int rs, int deg) {
    const bool ok = found && deg > 0;
    const Take k = take(&sh.n_out, ok ? 1 : 0);
    if (ok) {
      list[k.base + k.off] = entry_of(rs, deg);
      st_relaxed64(&out[k.base + k.off], entry_of(rs, deg));
    }
  }
};

// ---------------------------------------------- where a frontier's rows are --
struct ListSrc {
  const u64* list;
  unsigned n;
  __device__ __forceinline__ u64 get(unsigned group, int lane) const {
    const unsigned i = group * kWave + (unsigned)lane;
    return i < n ? list[i] : 0ull;
  }
};

struct QueueSrc {
  const SessShared& sh;
  const u64* q;
  unsigned pg;       // lane s: first group of segment s
  __device__ __forceinline__ u64 get(unsigned group, int lane) const {
    const int s = __popcll(__ballot(pg <= group)) - 1;
    const unsigned i = (group - (unsigned)__builtin_amdgcn_readlane((int)pg, s)) * kWave +
                       (unsigned)lane;
    return i < sh.p.seg_n[s] ? ld_relaxed(&q[(size_t)s * sh.p.stride + i]) : 0ull;
  }
};
__device__ __forceinline__ QueueSrc queue_src(const SessShared& sh, const u64* q) {
  const int lane = lane_id();
  return QueueSrc{sh, q, lane < kSessSegs ? sh.pre_g[lane] : ~0u};
}

// Claim up to E targets per lane, write their distances, hand their rows on.
// fresh: pull levels have rewritten the bitmap in this launch, so a stale line
// of it may hold anything; before that a stale word only lacks bits, and the
// claiming atomic decides.
template <int E, class Sink>
__device__ __forceinline__ void sess_visit(const SsspArgs& a, int L, u64* vis, bool fresh,
                                           const int* v, const bool* has, Sink& sink,
                                           SessCount& c) {
  bool claim[E];
  int rs[E], deg[E];
  if constexpr (E == 1) {
    // few edges a wave, so latency is everything: no look at the visited word
    // first, and the row bounds travel with the claim
    u64 old = ~0ull;
    int re = 0;
    rs[0] = 0;
    if (has[0]) {
      old = atom_or(&vis[v[0] >> 6], 1ull << (v[0] & 63));
      rs[0] = a.rp[v[0]];
      re = a.rp[v[0] + 1];
    }
    claim[0] = !((old >> (v[0] & 63)) & 1ull);
    deg[0] = re - rs[0];
    // the next level starts with this row: have its line on the way by then
    if (claim[0] && deg[0] > 0) c.ahead = a.col[rs[0]];
  } else {
    u64 w[E];
#pragma unroll
    for (int i = 0; i < E; ++i) w[i] = ~0ull;
    if (fresh) {
#pragma unroll
      for (int i = 0; i < E; ++i)
        if (has[i]) w[i] = ld_relaxed(&vis[v[i] >> 6]);
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i)
        if (has[i]) w[i] = vis[v[i] >> 6];
    }
#pragma unroll
    for (int i = 0; i < E; ++i)
      if (!((w[i] >> (v[i] & 63)) & 1ull)) w[i] = atom_or(&vis[v[i] >> 6], 1ull << (v[i] & 63));
#pragma unroll
    for (int i = 0; i < E; ++i) {
      claim[i] = !((w[i] >> (v[i] & 63)) & 1ull);
      rs[i] = deg[i] = 0;
      if (claim[i]) {
        rs[i] = a.rp[v[i]];
        deg[i] = a.rp[v[i] + 1] - rs[i];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (claim[i]) {
      a.dist[v[i]] = L;
      c.mf += (unsigned)deg[i];
    }
    c.nf += (unsigned)__popcll(__ballot(claim[i]));
    sink.add(claim[i], rs[i], deg[i]);
  }
}

// The frontier's groups of 64 rows dealt over `nwaves` waves, this one being
// gw; with fewer groups than waves, a group's steps over several waves.  A
// wave walks the union of its group's rows in steps of E x 64 edges.  Which
// row an edge belongs to: each row marks the step's slot of its first edge in
// LDS, and a maximum scan carries the marks on (a few LDS accesses a step,
// where a binary search by lane permutes took 36 for 256 edges).
template <int E, class Src, class Sink>
__device__ __forceinline__ void sess_push(const SsspArgs& a, int* own, int L, u64* vis,
                                          bool fresh, unsigned ngroups, unsigned gw, unsigned nwaves,
                                          const Src& src, Sink& sink, SessCount& c) {
  const int lane = lane_id();
  const unsigned split = max(nwaves / max(ngroups, 1u), 1u);
  for (unsigned vw = gw; vw < ngroups * split; vw += nwaves) {
    const unsigned part = vw / ngroups;
    const u64 ent = src.get(vw - part * ngroups, lane);
    const int deg = (int)(unsigned)(ent >> 32);
    const int incl = wave_incl_scan(deg);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int excl = incl - deg;
    const int first = (int)(unsigned)ent - excl;      // edge x of the union is col[first + x]
    for (int eb = (int)part * E * kWave; eb < total; eb += (int)split * E * kWave) {
#pragma unroll
      for (int q = 0; q < E; ++q) own[q * kWave + lane] = 0;
      wave_sync();
      if (deg > 0 && excl >= eb && excl < eb + E * kWave) own[excl - eb] = lane;
      wave_sync();
      // the row that covers the step's first edge
      int carry = 63 - __builtin_clzll(__ballot(deg > 0 && excl <= eb));
      int v[E];
      bool has[E];
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int x = eb + q * kWave + lane;
        const int o = wave_incl_max(max(own[q * kWave + lane], carry));
        carry = __builtin_amdgcn_readlane(o, kWave - 1);
        const int f = __shfl(first, o, kWave);
        has[q] = x < total;
        v[q] = has[q] ? a.col[f + x] : 0;
      }
      wave_sync();      // the marks are read before the next step clears them
      sess_visit<E>(a, L, vis, fresh, v, has, sink, c);
    }
  }
}

// One wave per bitmap word, a lane per unvisited node; the search is that of
// the level kernel's pull step.
template <class Sink>
__device__ __forceinline__ void sess_pull(const SsspArgs& a, int* rank_lane, int L, const u64* vin,
                                          u64* vout, unsigned gw, unsigned nwaves, Sink& sink,
                                          SessCount& c) {
  const int lane = lane_id();
  u64 nword = 0, nnoin = 0;
  if (gw < (unsigned)a.nw) {
    nword = ld_relaxed(&vin[gw]);
    nnoin = a.noin[gw];
  }
  for (unsigned w = gw; w < (unsigned)a.nw; w += nwaves) {
    const u64 word = nword;
    const u64 settled = word | nnoin;
    if (w + nwaves < (unsigned)a.nw) {
      nword = ld_relaxed(&vin[w + nwaves]);
      nnoin = a.noin[w + nwaves];
    }
    const int v = (int)(w * kWave) + lane;
    const int valid_n = min(kWave, a.n - (int)(w * kWave));
    const u64 full = valid_n >= kWave ? ~0ull : ((1ull << valid_n) - 1ull);
    if ((settled & full) == full) {
      if (lane == 0) st_relaxed64(&vout[w], word);
      continue;
    }
    bool found = false;
    int cur = 0, e = 0, rs = 0, deg = 0;
    const bool unvisited = lane < valid_n && !((settled >> lane) & 1ull);
    if (unvisited) {
      cur = a.ip[v];
      e = a.ip[v + 1];
      rs = a.rp[v];
      deg = a.rp[v + 1] - rs;
      const int lim = min(e, cur + a.lane_edges);
      for (; cur + 4 <= lim; cur += 4) {
        const int u0 = a.isrc[cur], u1 = a.isrc[cur + 1], u2 = a.isrc[cur + 2], u3 = a.isrc[cur + 3];
        const u64 b0 = ld_relaxed(&vin[u0 >> 6]) >> (u0 & 63);
        const u64 b1 = ld_relaxed(&vin[u1 >> 6]) >> (u1 & 63);
        const u64 b2 = ld_relaxed(&vin[u2 >> 6]) >> (u2 & 63);
        const u64 b3 = ld_relaxed(&vin[u3 >> 6]) >> (u3 & 63);
        c.edges += 4;
        if ((b0 | b1 | b2 | b3) & 1ull) {
          found = true;
          break;
        }
      }
      for (; !found && cur < lim; ++cur) {
        const int u = a.isrc[cur];
        c.edges += 1;
        if ((ld_relaxed(&vin[u >> 6]) >> (u & 63)) & 1ull) found = true;
      }
    }
    bool searching = unvisited && !found && cur < e;
    u64 um = __ballot(searching);
    while (um) {
      const int cnt = __popcll(um);
      const int rank = __popcll(um & lanes_below());
      if (searching) rank_lane[rank] = lane;
      wave_sync();
      const int owner = rank_lane[lane % cnt];
      const int off = lane / cnt;
      const int oc = __shfl(cur, owner, kWave);
      const int oe = __shfl(e, owner, kWave);
      const int idx = oc + off;
      bool hit = false;
      if (idx < oe) {
        const int u = a.isrc[idx];
        c.edges += 1;
        hit = (ld_relaxed(&vin[u >> 6]) >> (u & 63)) & 1ull;
      }
      const u64 hm = __ballot(hit);
      u64 fold = 0;
      for (int sft = 0; sft < kWave; sft += cnt) fold |= hm >> sft;
      wave_sync();
      if (searching) {
        if ((fold >> rank) & 1ull) found = true;
        cur += (kWave - rank + cnt - 1) / cnt;
        searching = !found && cur < e;
      }
      um = __ballot(searching);
    }
    const u64 newbits = __ballot(found);
    if (lane == 0) st_relaxed64(&vout[w], word | newbits);
    if (newbits) {
      if (found) {
        a.dist[v] = L;
        c.mf += (unsigned)deg;
      }
      c.nf += (unsigned)__popcll(newbits);
      sink.add(found, rs, deg);
    }
  }
}

// Per-wave counters to the workgroup's.
__device__ __forceinline__ void add_counts(SessShared& sh, const SessCount& c, bool pull) {
  const unsigned mf = wave_sum(c.mf);
  const unsigned ed = pull ? wave_sum(c.edges) : 0u;
  if (lane_id() == 0 && (c.nf | ed)) {
    atomicAdd(&sh.nf, c.nf);
    atomicAdd(&sh.mf, mf);
    if (ed) atomicAdd(&sh.edges, ed);
  }
}

// A grid or cluster level's own step.
template <class Sink>
__device__ __forceinline__ void sess_step(const SsspArgs& a, const SessArgs& x, SessShared& sh,
                                          Sink& sink, SessCount& c) {
  const int wv = threadIdx.x / kWave;
  const SessPlan& p = sh.p;
  const int L = (int)uniform(p.level);
  const unsigned K = uniform(p.K);
  const unsigned nwaves = K * kSW;
  // neighbouring groups to different compute units
  const unsigned gw = (unsigned)wv * K + sh.rank;
  const bool cur = uniform(p.cur) != 0;
  u64* vcur = cur ? a.vis1 : a.vis0;
  if (uniform(p.pull)) {
    sess_pull(a, sh.own[wv], L, vcur, cur ? a.vis0 : a.vis1, gw, nwaves, sink, c);
    return;
  }
  const QueueSrc src = queue_src(sh, x.q[p.qp]);
  const unsigned ngroups = uniform(sh.pre_g[kSessSegs]);
  const bool fresh = uniform(p.pull_levels) > 0;
  // with at most two steps of 64 edges a wave, short steps
  if (uniform(p.fe) <= nwaves * 2 * kWave)
    sess_push<1>(a, sh.own[wv], L, vcur, fresh, ngroups, gw, nwaves, src, sink, c);
  else
    sess_push<4>(a, sh.own[wv], L, vcur, fresh, ngroups, gw, nwaves, src, sink, c);
}

// ---------------------------------------------------------------- grid level --
// Runs the level, then the barrier.  Returns the next record's number (0: a
// wait timed out).
__device__ __forceinline__ unsigned grid_level(const SsspArgs& a, const SessArgs& x,
                                               SessShared& sh, unsigned gen) {
  const int t = threadIdx.x, lane = lane_id();
  SessCtrl* sc = x.sc;
  SessSlot* slot = &sc->slot[gen % 3];
  const unsigned stripe = sh.rank % kSessStripes;
  u64* qout = x.q[sh.p.qp ^ 1] + (size_t)stripe * x.qcap;
  unsigned* qn = &slot->q[stripe].n;
  const bool pull = sh.p.pull != 0;
  {
    SessCount c{0, 0, 0, 0};
    PieceSink<false> sink{sh, qout, qout, qn, (unsigned)kStage};
    sess_step(a, x, sh, sink, c);
    add_counts(sh, c, pull);
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
      const unsigned v = lane == 0 ? sh.nf : lane == 1 ? sh.mf : sh.edges;
      atom_add(&slot->grp[grp].w[lane], (1ull << 48) | v);
    }
    wave_sync();
    if (lane == 0) sh.nf = sh.mf = sh.edges = sh.n_out = 0;
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
        const u64 ed = pull ? wave_sum(w2 & low) : (u64)sh.p.fe;
        const LevelState st = sess_decide(a, sh.p, SlotSum{(unsigned)nf, mf, ed}, true);
        set_segments(sh, sq);
        sess_plan(a, sh.p, st, mf, sh.members);
        if (lane == 0) {
          sh.p.qp ^= 1;
          sh.p.stride = x.qcap;
        }
        sess_publish(sc, sh, gen + 1);
        next = gen + 1;
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
// parity, tagged with the level) and reads all of them, so each holds the
// level's sums and takes the same decision.  A member cannot be two levels
// ahead of another, so two lines do.  On return sh holds the next level's
// plan, which only workgroup 0 uses; the others take it from the next record.
// Returns false if a wait timed out.
__device__ __forceinline__ bool cluster_run(const SsspArgs& a, const SessArgs& x, SessShared& sh) {
  const int t = threadIdx.x, lane = lane_id();
  SessCtrl* sc = x.sc;
  for (;;) {
    const unsigned L = uniform(sh.p.level);
    const bool pull = uniform(sh.p.pull) != 0;
    // the counter of the next level was last read before this one began
    if (sh.rank == 0 && t == 0) st_relaxed(&sc->over[(L + 1) % 3].n, 0u);
    {
      SessCount c{0, 0, 0, 0};
      u64* qout = x.q[sh.p.qp ^ 1];
      PieceSink<true> sink{sh, qout + (size_t)sh.rank * x.ccap,
                           qout + (size_t)kSessGroup * x.ccap, &sc->over[L % 3].n, x.ccap};
      sess_step(a, x, sh, sink, c);
      add_counts(sh, c, pull);
      keep(c.ahead);
    }
    wait_all();
    __syncthreads();
    if (t < kWave) {
      const unsigned n = sh.n_out;
      const unsigned mine = lane == 0 ? n : lane == 1 ? sh.nf : lane == 2 ? sh.mf : sh.edges;
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
        const u64 ed = pull ? (u64)wave_sum(mem ? (unsigned)w3 : 0u) : (u64)sh.p.fe;
        unsigned seg = min(cnt, x.ccap);
        if (__ballot(cnt > x.ccap)) {
          const unsigned ov = ld_relaxed(&sc->over[L % 3].n);
          if (lane == kSessGroup) seg = ov;
        }
        const LevelState st = sess_decide(a, sh.p, SlotSum{(unsigned)nf, mf, ed}, sh.rank == 0);
        set_segments(sh, seg);
        sess_plan(a, sh.p, st, mf, sh.members);
        if (lane == 0) {
          sh.nf = sh.mf = sh.edges = sh.n_out = 0;
          sh.p.qp ^= 1;
          sh.p.stride = x.ccap;
        }
      }
      if (lane == 0) sh.ok = state;
    }
    __syncthreads();
    if (sh.ok != 1) return sh.ok == 2;
    if (sh.p.mode != kModeCluster) {
      // clear for the next run, which starts with a record of workgroup 0
      // after its next wait for its stores
      if (sh.rank == 0 && t < 3) st_relaxed(&sc->over[t].n, 0u);
      return true;
    }
  }
}

// ---------------------------------------------------------------- solo levels --
// Workgroup 0 alone.  On entry `cur` holds ncur rows and sh.p the level to run;
// on return sh.p is the next level, its queue written, or the end.
__device__ __forceinline__ void solo_run(const SsspArgs& a, const SessArgs& x, SessShared& sh,
                                         u64* cur, unsigned ncur) {
  const int t = threadIdx.x, wv = t / kWave, lane = lane_id();
  int ahead = 0;
  for (;;) {
    u64* nxt = cur == sh.stage ? sh.stage + kSoloCap : sh.stage;
    {
      SessCount c{0, 0, 0, 0};
      ListSink sink{sh, nxt, x.q[sh.p.qp ^ 1]};
      sess_push<1>(a, sh.own[wv], (int)uniform(sh.p.level), uniform(sh.p.cur) ? a.vis1 : a.vis0,
                   true, (ncur + kWave - 1) / kWave, (unsigned)wv, (unsigned)kSW,
                   ListSrc{cur, ncur}, sink, c);
      add_counts(sh, c, false);
      keep(ahead);        // (of the level before)
      ahead = c.ahead;
      if (wv == kSW - 1 && !sh.p.full) {
        // the wave that is first out of work looks who has joined
        const u64 w = lane < kSessGroups ? ld_relaxed(&x.sc->joined[lane].w) : 0ull;
        const unsigned cnt = wave_sum((unsigned)__popcll(w));
        if (lane == 0 && cnt + 1 >= gridDim.x) sh.p.full = 1;
      }
    }
    __syncthreads();
    ncur = uniform(sh.n_out);
    cur = nxt;
    if (t < kWave) {
      const u64 mf = uniform(sh.mf);
      const LevelState st = sess_decide(a, sh.p, SlotSum{uniform(sh.nf), mf, sh.p.fe}, true);
      const bool solo = is_solo(a, st, mf);
      if (!solo) {
        set_segments(sh, lane == 0 ? ncur : 0u);
      }
      sess_plan(a, sh.p, st, mf, sh.members);
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

// 4 waves per SIMD: asking for 5, 6 or 8 spills registers and is slower
// (R-MAT 20: 2.09, 2.20, 2.14 and 2.36 ms per 16 sources when measured).
__global__ __launch_bounds__(kSB, 4) void sssp_session(SsspArgs a, SessArgs x) {
  __shared__ SessShared sh;
  const unsigned long long t_start = wall_clock64();
  const int t = threadIdx.x, lane = lane_id();
  const unsigned bid = blockIdx.x;
  SessCtrl* sc = x.sc;
  // consecutive workgroups go to the 8 XCDs in turn: word (layer, XCD), bit =
  // position on that XCD, so that 32 consecutive ranks share an XCD's L2
  const unsigned wi = (bid >> 8) * 8 + (bid & 7), bi = (bid >> 3) & 31;
  if (t == 0) {
    sh.nf = sh.mf = sh.edges = sh.n_out = 0;
    sh.ok = 1;
    if (bid != 0 && (atom_or(&sc->joined[wi].w, 1ull << bi) & kClosed)) sh.ok = 0;
  }
  // the rank if every workgroup joins
  if (t < kWave) sess_rank(launch_word(lane, gridDim.x), sh, wi, bi);
  __syncthreads();
  if (!sh.ok) return;
  unsigned gen = 0;
  bool ranked = false, lead = false;    // lead: workgroup 0 holds the next plan
  if (bid == 0) {
    // level 0: the source, a queue of one row
    const int s = x.source;
    const int rs = a.rp[s], deg = a.rp[s + 1] - rs;
    if (t < kWave) {
      SessPlan& p = sh.p;
      if (lane == 0) {
        p.level = p.cur = p.pull = 0;
        p.mu = (unsigned)a.m;
        p.last_nonempty = p.push_levels = p.pull_levels = p.prev_nf = 0;
        p.edges_lo = p.edges_hi = p.source_edges = p.reached = 0;
        p.qp = 0;
        p.stride = x.qcap;
        p.full = 0;
        if (a.lrec > 0) a.level_dir[0] = 0;
        sh.stage[0] = entry_of(rs, deg);
        st_relaxed64(&x.q[0][0], entry_of(rs, deg));
      }
      wave_sync();
      const LevelState st = sess_decide(a, p, SlotSum{1u, (u64)deg, 0}, true);
      set_segments(sh, lane == 0 ? 1u : 0u);
      sess_plan(a, p, st, (u64)deg, 1u);
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
      // close the member list the first time, then publish the plan
      if (t < kWave) {
        if (!sh.p.done && !ranked) {
          bool full = sh.p.full != 0;
          while (!full) {
            const u64 w = lane < kSessGroups ? ld_relaxed(&sc->joined[lane].w) : 0ull;
            const unsigned cnt = wave_sum((unsigned)__popcll(w));
            full = cnt + 1 >= gridDim.x;
            if (wall_clock64() - t_start > kJoinTicks) break;
          }
          if (!full) {
            unsigned w = 0;
            if (lane < kSessGroups) {
              w = (unsigned)atom_or(&sc->joined[lane].w, kClosed);
              if (lane == 0) w |= 1u;
              st_relaxed(&sc->memb[lane], w);
            }
            sess_rank(w, sh, 0, 0);
            wait_all();
          }
          if (lane == 0) sh.p.full = full ? 1 : 0;
          wave_sync();
          // the plan was made without knowing the members
          LevelState st = sess_state(sh.p);
          sess_plan(a, sh.p, st, sh.p.fe, sh.members);
        }
        sess_publish(sc, sh, gen + 1);
      }
      ranked = ranked || !sh.p.done;
      gen += 1;
      lead = false;
      __syncthreads();
    }
    if (sh.p.mode == kModeEnd) return;
    if (!ranked) {
      if (!sh.p.full) {
        __syncthreads();
        if (t < kWave)
          sess_rank(lane < kSessGroups ? ld_relaxed(&sc->memb[lane]) : 0u, sh, wi, bi);
        __syncthreads();
      }
      ranked = true;
    }
    const bool mine = sh.p.mode == kModeSolo ? bid == 0 : sh.rank < sh.p.K;
    bool poll = !mine;
    if (mine && sh.p.mode == kModeGrid) {
      gen = grid_level(a, x, sh, gen);
      if (!gen) return;
    } else if (mine) {
      if (sh.p.mode == kModeCluster) {
        if (!cluster_run(a, x, sh)) return;
        poll = bid != 0;
        lead = bid == 0;
      }
      if (bid == 0 && sh.p.mode == kModeSolo) {
        // the frontier from the queue: at most kSoloCap rows
        __syncthreads();
        const QueueSrc src = queue_src(sh, x.q[sh.p.qp]);
        for (unsigned g = (unsigned)(t / kWave); g < sh.pre_g[kSessSegs]; g += kSW) {
          const u64 e = src.get(g, lane);
          const Take k = take(&sh.n_out, e ? 1 : 0);
          if (e && k.base + k.off < (unsigned)kSoloCap) sh.stage[k.base + k.off] = e;
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

// dist = -1 except dist[source] = 0, visited = {source}, control block clear.
__global__ __launch_bounds__(kSB) void sess_init(SsspArgs a, SessArgs x) {
  const unsigned tid = blockIdx.x * kSB + threadIdx.x, nt = gridDim.x * kSB;
  if (tid == 0) {
    if (a.hm) a.hm->t_start = wall_clock64();
    a.ctrl->st[1].done = 0;
  }
  const int s = x.source;
  u64* c = reinterpret_cast<u64*>(x.sc);
  for (unsigned i = tid; i < sizeof(SessCtrl) / 8; i += nt) c[i] = 0;
  for (unsigned w = tid; w < (unsigned)a.nw; w += nt)
    a.vis0[w] = (int)w == (s >> 6) ? (1ull << (s & 63)) : 0ull;
  for (unsigned i = tid; i < (unsigned)a.n; i += nt) a.dist[i] = (int)i == s ? 0 : -1;
}

// After the session: its writes are complete, the end goes to the host.
__global__ __launch_bounds__(kWave) void sess_close(SsspArgs a) {
  if (threadIdx.x != 0) return;
  LevelState st = a.ctrl->st[1];
  if (!st.done) st.done = 2;       // a wait timed out
  report(a, 1, st, true);
}

// ------------------------------------------------------------------ host --
dawn_status sess_launch(Ctx* ctx, const SsspArgs& a, const SessArgs& x, int blocks_per_cu,
                        hipStream_t s) {
  static std::atomic<int> occ_cache{0};
  int occ = occ_cache.load(std::memory_order_relaxed);
  if (!occ) {
    DAWN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, sssp_session, kSB, 0));
    occ = std::max(occ, 1);
    occ_cache.store(occ, std::memory_order_relaxed);
  }
  const int per_cu = std::min(blocks_per_cu > 0 ? blocks_per_cu : kSessPerCu, occ);
  // no more workgroups than a level of this graph can use
  const long long useful = std::max<long long>((a.nw + kSW - 1) / kSW,
                                               (a.m + kEdgesPerWg - 1) / kEdgesPerWg);
  const int grid = (int)std::max<long long>(
      1, std::min<long long>({useful, (long long)per_cu * ctx->num_cu,
                              (long long)kSessGroups * kSessGroup}));
  const int fill = std::max(1, std::min((a.n + kSB - 1) / kSB, ctx->num_cu * 4));
  hipLaunchKernelGGL(sess_init, dim3(fill), dim3(kSB), 0, s, a, x);
  hipLaunchKernelGGL(sssp_session, dim3(grid), dim3(kSB), 0, s, a, x);
  hipLaunchKernelGGL(sess_close, dim3(1), dim3(kWave), 0, s, a);
  DAWN_HIP(hipGetLastError());
  return DAWN_OK;
}

}  // namespace dawn
