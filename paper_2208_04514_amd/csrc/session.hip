// Single-source traversal in one launch (session_dev.hpp), by hops.
//
// The level step is the one of sssp.hip (push: Section 3.3, Algorithm 2; pull:
// Section 3.2, Algorithm 1 with the early exit).  What differs is where a level
// ends.  A launch per level costs about 10 us even when the level has a few
// hundred edges (dispatch, first reads of a state the other XCDs wrote, the
// write-back at the end), and most levels of a road-like graph, and the first
// and last of any graph, are that small.  Distances are plain stores nothing
// reads before the launch has ended; the launch after it reports the end.
//
// Bound: a level's chain of dependent memory round trips (queue entry, targets,
// claim with the row bounds, queue store, report), about 2 us solo, 4.5 in a
// cluster, 7 in the grid, until a level has some 10^5 edges; from there the
// claims and bitmap reads.  Per source against a launch per level (MI355X):
// R-MAT 20 186 -> 95 us; grid 2048^2 (some 130 levels) 2.64 -> 1.41 ms; grid
// 1023 x 1025 without shortcuts (some 1,500 levels) 17.3 -> 6.5 ms; uniform
// n = 4096 70 -> 51 us.
#include <string.h>

#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"
#include "session_dev.hpp"
#include "sssp_dev.hpp"

namespace dawn {

__device__ __forceinline__ u64 entry_of(int rs, int deg) {
  return (u64)(unsigned)rs | ((u64)(unsigned)deg << 32);
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
        c.scan += 4;
        if ((b0 | b1 | b2 | b3) & 1ull) {
          found = true;
          break;
        }
      }
      for (; !found && cur < lim; ++cur) {
        const int u = a.isrc[cur];
        c.scan += 1;
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
        c.scan += 1;
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

// Queue entries are (row start, out-degree).
struct HopPolicy {
  static constexpr int kPiece = kHopPiece;
  static constexpr bool kAdmits = true;
  template <class Plan>
  static __device__ __forceinline__ unsigned long long join_ticks(const Plan& p, int words) {
    return admit_ticks(p, words);
  }
  using Args = SsspArgs;
  // LevelState's fields
  struct State {
    unsigned level, cur, pull, done;
    unsigned mu, last_nonempty, push_levels, pull_levels, prev_nf;
    unsigned edges_lo, edges_hi, source_edges, reached;
  };
  using Shared = SessShared<HopPolicy>;

  static __device__ __forceinline__ u64 entry(int rs, int deg, int i) {
    return entry_of(rs + i * kPiece, min(kPiece, deg - i * kPiece));
  }
  static __device__ __forceinline__ u64 row_entry(int rs, int deg) { return entry_of(rs, deg); }
  static __device__ __forceinline__ int words(const SsspArgs& a) { return a.nw; }
  static __device__ __forceinline__ bool scans(const SessPlan<State>& p) { return p.u.pull != 0; }

  template <int E, class Src, class Sink>
  static __device__ __forceinline__ void push(const SsspArgs& a, int* own, int L, u64* vis,
                                              bool fresh, unsigned ngroups, unsigned gw,
                                              unsigned nwaves, const Src& src, Sink& sink,
                                              SessCount& c) {
    walk_rows<E>(
        own, ngroups, gw, nwaves, src,
        [](u64 e, unsigned, int& rs, int& deg) {
          if (e == kNoEntry) return;
          rs = (int)(unsigned)e;
          deg = (int)(unsigned)(e >> 32);
        },
        [&](const int*, const int* at, const bool* has) {
          int v[E];
#pragma unroll
          for (int q = 0; q < E; ++q) v[q] = has[q] ? a.col[at[q]] : 0;
          sess_visit<E>(a, L, vis, fresh, v, has, sink, c);
        });
  }

  template <class Sink>
  static __device__ __forceinline__ void step(const SsspArgs& a, const SessArgs& x, Shared& sh,
                                              Sink& sink, SessCount& c) {
    const int wv = threadIdx.x / kWave;
    const State& u = sh.p.u;
    const int L = (int)uniform(u.level);
    const unsigned K = uniform(sh.p.K);
    const unsigned nwaves = K * kSW;
    // neighbouring groups to different compute units
    const unsigned gw = (unsigned)wv * K + sh.rank;
    const bool cur = uniform(u.cur) != 0;
    u64* vcur = cur ? a.vis1 : a.vis0;
    if (uniform(u.pull)) {
      sess_pull(a, sh.own[wv], L, vcur, cur ? a.vis0 : a.vis1, gw, nwaves, sink, c);
      return;
    }
    const QueueSrc<HopPolicy> src = queue_src(sh, x.q[sh.p.qp]);
    const unsigned ngroups = uniform(sh.pre_g[kSessSegs]);
    const bool fresh = uniform(u.pull_levels) > 0;
    // with at most two steps of 64 edges a wave, short steps
    if (uniform(sh.p.fe) <= nwaves * 2 * kWave)
      push<1>(a, sh.own[wv], L, vcur, fresh, ngroups, gw, nwaves, src, sink, c);
    else
      push<4>(a, sh.own[wv], L, vcur, fresh, ngroups, gw, nwaves, src, sink, c);
  }

  template <class Sink>
  static __device__ __forceinline__ void solo(const SsspArgs& a, Shared& sh, const u64* cur,
                                              unsigned ncur, Sink& sink, SessCount& c) {
    const int wv = threadIdx.x / kWave;
    push<1>(a, sh.own[wv], (int)uniform(sh.p.u.level), uniform(sh.p.u.cur) ? a.vis1 : a.vis0, true,
            (ncur + kWave - 1) / kWave, (unsigned)wv, (unsigned)kSW, ListSrc{cur, ncur}, sink, c);
  }

  // Fold the level's counters into the state and choose the next level.  Every
  // lane of wave 0 computes the same.  A pull level has made the other bitmap
  // the current one.
  static __device__ __forceinline__ void advance(const SsspArgs& a, Shared& sh, unsigned nf, u64 mf,
                                                 u64 examined, bool record) {
    State& u = sh.p.u;
    LevelState st;
    st.level = (int)u.level;
    st.cur = (int)(u.cur ^ u.pull);
    st.pull = (int)u.pull;
    st.done = 0;
    st.mu = (long long)u.mu;
    st.last_nonempty = (int)u.last_nonempty;
    st.push_levels = (int)u.push_levels;
    st.pull_levels = (int)u.pull_levels;
    st.launches = 1;
    st.prev_nf = u.prev_nf;
    st.mbar = 0;
    st.edges_total = (u64)u.edges_lo | ((u64)u.edges_hi << 32);
    st.source_edges = u.source_edges;
    st.reached = u.reached;
    // a push level examines every out-edge of its frontier
    const SlotSum sum{nf, mf, u.pull ? examined : (u64)sh.p.fe};
    decide(a, st, sum, record && lane_id() == 0);
    set_plan<HopPolicy>(sh, st.done != 0, st.pull != 0, mf, a.nw, a.small_edges);
    if (lane_id() == 0) {
      u.level = (unsigned)st.level;
      u.cur = (unsigned)st.cur;
      u.pull = (unsigned)st.pull;
      u.done = (unsigned)st.done;
      u.mu = (unsigned)st.mu;
      u.last_nonempty = (unsigned)st.last_nonempty;
      u.push_levels = (unsigned)st.push_levels;
      u.pull_levels = (unsigned)st.pull_levels;
      u.prev_nf = st.prev_nf;
      u.edges_lo = (unsigned)st.edges_total;
      u.edges_hi = (unsigned)(st.edges_total >> 32);
      u.source_edges = (unsigned)st.source_edges;
      u.reached = (unsigned)st.reached;
      if (st.done) a.ctrl->st[1] = st;
    }
  }

  static __device__ __forceinline__ void begin(const SsspArgs& a, const SessArgs& x, Shared& sh) {
    const int s = x.source;
    const int rs = a.rp[s], deg = a.rp[s + 1] - rs;
    if (lane_id() == 0) {
      State& u = sh.p.u;
      u.level = u.cur = u.pull = u.done = 0;
      u.mu = (unsigned)a.m;
      u.last_nonempty = u.push_levels = u.pull_levels = u.prev_nf = 0;
      u.edges_lo = u.edges_hi = u.source_edges = u.reached = 0;
      sh.p.fe = 0;
      if (a.lrec > 0) a.level_dir[0] = 0;
      sh.stage[0] = entry_of(rs, deg);
      st_relaxed64(&x.q[0][0], entry_of(rs, deg));
    }
    wave_sync();
    advance(a, sh, 1u, (u64)deg, 0ull, true);     // level 0: the source
  }
};

// 4 waves per SIMD: asking for 5, 6 or 8 spills registers and is slower
// (R-MAT 20: 2.09, 2.20, 2.14 and 2.36 ms per 16 sources when measured).
__global__ __launch_bounds__(kSB, 4) void sssp_session(SsspArgs a, SessArgs x) {
  __shared__ SessShared<HopPolicy> sh;
  session<HopPolicy>(a, x, sh);
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
  const int grid = sess_grid(ctx, per_cu, blocks_per_cu > 0 ? 1 : ctx_share(ctx), a.nw, a.m);
  // (the control block in one go)
  constexpr int least = (int)((sizeof(SessCtrl) / 8 + kSB - 1) / kSB);
  const int fill = std::max(least, std::min((a.n + kSB - 1) / kSB, ctx->num_cu * 4));
  hipLaunchKernelGGL(sess_init, dim3(fill), dim3(kSB), 0, s, a, x);
  hipLaunchKernelGGL(sssp_session, dim3(grid), dim3(kSB), 0, s, a, x);
  hipLaunchKernelGGL(sess_close, dim3(1), dim3(kWave), 0, s, a);
  DAWN_HIP(hipGetLastError());
  return DAWN_OK;
}

}  // namespace dawn
