// Weighted single-source shortest paths: DAWN's level loop over the (min, +)
// semiring.
//
// The paper closes (Section 5) by naming weighted graphs, through the same
// vector-matrix step over (min, +) instead of (OR, AND), as future work.  Here
// that step is the SOVM of Algorithm 2 with the Boolean union replaced by a
// minimum of sums: a round takes the nodes whose distance dropped in the
// previous round (the frontier), and for every out-edge (u, v, w) lowers
// dist[v] to dist[u] + w with an atomic minimum; the nodes whose distance
// dropped form the next frontier.  With non-negative weights the loop stops
// at the fixed point dist[v] = min over in-edges of dist[u] + w, which is the
// shortest-path distance (the Bellman-Ford argument: after k rounds every
// shortest path of at most k edges is exact; a frontier node's edges are
// relaxed again whenever its distance drops).  Unlike the Boolean loop a
// node may join several frontiers, so rounds can outnumber BFS levels.
//
// Order.  Relaxing in hop order alone relaxes an edge again whenever its source
// improves: 3 times on R-MAT 20, 7 on a road-like grid (weights 1..100).  So
// distances are settled in buckets of width delta, the near-far form of
// delta-stepping (Meyer and Sanders): only nodes below the bucket's bound T join
// the frontier; when it is empty every distance below T is final, and one pass
// over the distances collects the next bucket's nodes.  With delta below the
// largest weight (`split`), a round also leaves alone the edges that reach past
// T, and they are relaxed once, from the settled distances, when the bucket is
// done.  For that the weights come with a copy of the rows whose edges lighter
// than delta stand first: a round looks at those alone.  The settled nodes have
// a bitmap, which most targets of the later pass are found in (it stays in the
// caches; distances at random do not).  No bucket is empty, however far apart distances
// lie, so the levels are bounded by the nodes (max_rounds): a collection counts the
// nodes less than delta past its bucket, and where there is none the next bucket is the
// one with the smallest distance further on, or that the relaxations past T make.
//
// delta = kDelta x mean weight / mean out-degree: the denser the graph, the
// more often an unsettled node's row is relaxed in vain, the sparser, the fewer
// nodes a round has to work on.
//
// Bound: on R-MAT 20 the rounds over hubs' rows (random distances, several
// dependent accesses an edge: 30 to 120 G edges/s), on grids the levels' chains
// (5 to 8 us each).  Per source (MI355X, weights 1..100), hop order with a
// launch per round -> now: R-MAT 20 1.74 -> 1.00 ms, grid 1024^2 4.6 -> 1.7 ms.
//
// Distances are int32 with -1 for "unreached": compared as unsigned, -1 is
// the largest value, so the atomic minimum needs no sentinel pass.  The
// upload of the weights checks that every path length fits (max weight x
// (n - 1) < 2^31 - 1).
//
// All rounds run in one launch (session_dev.hpp).  A node joins the next
// frontier once per round: its bit in the next round's membership bitmap is
// set with an atomic OR, and each round clears the bits of the frontier it
// consumes, so the bitmap of parity p is clear again when it is next written,
// but for nodes that dropped without an edge to relax: those are in no queue, and
// their bits stay until the init kernel of the next run clears both bitmaps.
// (Within a run nothing is lost by it: such a node drops again only in the same
// bucket, where it still has no edge to relax.)
#include <string.h>

#include <algorithm>
#include <vector>

#include "device_util.hpp"
#include "internal.hpp"
#include "session_dev.hpp"

namespace dawn {

// Bucket width, measured at 8, 16, 32 and 64 (ms, 4 sources R-MAT 20: 4.51,
// 4.52, 5.85, 7.45; 2 sources grid 1024^2: 4.44, 3.68, 3.38, 3.34; a smaller
// grid 2.04, 1.82, 1.85, 1.95): the narrower where the light rows pay (split).
constexpr double kDelta = 16.0;
constexpr double kDeltaWhole = 32.0;
// A bucket whose nodes have fewer out-edges than this takes some 25 us whatever
// it holds: the next is twice as wide, once half of the graph's edges are settled.
constexpr unsigned kSmallBucket = 1 << 19;
// So it is after this many buckets of one workgroup's work in a row: a long path of
// heavy edges then takes one level a node and not four.  (A path of 2000 edges of
// weight 100 before a clique: 22 ms without this, 6.1 with; a round a launch 16.)
constexpr unsigned kThinBuckets = 16;

// What a weighted run leaves for the host (coherent host memory).
struct WMirror {
  unsigned rounds, done;
  unsigned long long reached, source_edges;
  unsigned long long t_start, t_end;
  unsigned end_tag;
};

struct WCtrl {
  SessCtrl sess;
  alignas(kLine) unsigned done;         // 1 finished, 2 watchdog
  unsigned rounds;
  // the closing reduction, a line per stripe: reached nodes, their out-degrees
  struct alignas(kLine) Part {
    u64 reached, edges;
  } part[kStripes];
  alignas(kLine) unsigned closed;       // workgroups that have added theirs
  // kFar - the smallest distance past the bucket that a level came upon (0: none), by
  // barrier group; three, used in turn
  struct alignas(kLine) Low {
    int v;
  } low[3][kSessGroups];
};

struct WArgs {
  int32_t n;
  int32_t nw;
  const int32_t* rp;
  const int32_t* col;
  const int32_t* wt;            // weight of each CSR entry
  const int32_t* light;         // split: a row's edges lighter than delta stand first, this
                                //   many of them (null: rows as uploaded)
  int32_t* dist;                // output (device)
  u64* fin;                     // split: nodes of finished buckets
  u64* inq[2];                  // frontier membership bitmaps by round parity
  WCtrl* ctrl;
  WMirror* hm;
  unsigned seq;
  unsigned delta;               // bucket width
  int32_t split;                // delta < largest weight: edges past the bound wait
  unsigned half;                // half the graph's edges
  unsigned max_rounds;
};

__device__ __forceinline__ unsigned umin_atomic(int32_t* p, unsigned v) {
  return __hip_atomic_fetch_min(reinterpret_cast<unsigned*>(p), v, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

constexpr unsigned kUnreached = ~0u;
constexpr int kFar = 0x7fffffff;        // larger than any distance
constexpr unsigned kWhole = ~0u;        // piece number of an uncut row

// What a level of the session does.
enum WPhase {
  kNear = 0,        // relax the frontier's rows; targets below the bound join the next
  kSettled = 1,     // collect the bucket's nodes
  kHeavy = 2,       // relax their edges that reach the bound or past it
  // from here on the smallest distance past the bucket may be wanted
  kCollect = 3,     // collect the nodes of the next bucket
  kHeavyGap = 4     // kHeavy, where no node was less than delta past the bucket
};

// Queue entries are (node, piece of its row).
struct WeightPolicy {
  static constexpr int kPiece = kWeightPiece;
  static constexpr bool kAdmits = true;
  template <class Plan>
  static __device__ __forceinline__ unsigned long long join_ticks(const Plan& p, int words) {
    return admit_ticks(p, words);
  }
  using Args = WArgs;
  struct State {
    unsigned phase, par;        // par: membership bitmap of the frontier
    unsigned lo, hi;            // the bucket: distances in [lo, hi)
    unsigned width;             // of the next collection
    unsigned rounds;            // near rounds run
    unsigned far;               // kFar - a bound below the next distance (0: none left)
    unsigned gap;               // no node was less than delta past the bucket
    unsigned lows;              // levels that used WCtrl::low so far
    unsigned settled;           // out-edges of the finished buckets
    unsigned thin;              // buckets of one workgroup's work in a row
    unsigned steps;
  };
  struct Shared : SessShared<WeightPolicy> {
    int low;                    // this workgroup's part of WCtrl::low
  };
  using S = SessShared<WeightPolicy>;

  static __device__ __forceinline__ u64 entry(int v, int, int i) {
    return (u64)(unsigned)v | ((u64)(unsigned)i << 32);
  }
  static __device__ __forceinline__ u64 row_entry(int v, int) {
    return (u64)(unsigned)v | ((u64)kWhole << 32);
  }
  static __device__ __forceinline__ int words(const WArgs& a) { return a.nw; }
  static __device__ __forceinline__ bool scans(const SessPlan<State>& p) { return p.scan != 0; }

  // Relax up to E edges per lane.  near: targets that drop below hi join the
  // next frontier; with `split`, edges of the other kind are left alone.
  template <int E, class Sink>
  static __device__ __forceinline__ void relax(const WArgs& a, bool near, bool lite, unsigned hi, u64* next,
                                               const int* v, const unsigned* cand, const bool* has0,
                                               Sink& sink, SessCount& c) {
    unsigned cur[E];
    bool go[E], has[E];
#pragma unroll
    for (int i = 0; i < E; ++i) has[i] = has0[i];
    if (E > 1 && a.split) {
      // (a stale word lacks bits, no more)
      u64 f[E];
#pragma unroll
      for (int i = 0; i < E; ++i) f[i] = has[i] ? a.fin[v[i] >> 6] : 0ull;
#pragma unroll
      for (int i = 0; i < E; ++i) has[i] = has[i] && !((f[i] >> (v[i] & 63)) & 1ull);
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
      // (the distance as it is now: an older, larger one would cost an atomic,
      // and those on a hub's line run one after another)
      cur[i] = 0;
      if (has[i]) cur[i] = (unsigned)ld_relaxed(&a.dist[v[i]]);
    }
    if constexpr (E == 1) {
      // latency: the claim of the frontier bit travels with the minimum.  If
      // another relaxation got there first, v has dropped in this round all the
      // same and belongs in the next frontier.
      go[0] = has[0] && cand[0] < cur[0];
      bool first = false;
      int deg = 0;
      if (go[0]) {
        const u64 bit = 1ull << (v[0] & 63);
        umin_atomic(&a.dist[v[0]], cand[0]);
        if (near && cand[0] < hi) {
          first = !(atom_or(&next[v[0] >> 6], bit) & bit);
          deg = near_degree(a, lite, v[0]);
        }
        if (!near) c.low = max(c.low, kFar - (int)cand[0]);
      }
      put(first, v[0], deg, sink, c);
    } else {
      if (!near) {
        // (whether another relaxation got there first is not asked: its candidate is the
        // smaller then, and the minimum the same.  R-MAT 20's heavy levels take 331 us a
        // source with atomics that return the old distance, 295 so)
#pragma unroll
        for (int i = 0; i < E; ++i) {
          if (has[i] && cand[i] < cur[i]) {
            umin_atomic(&a.dist[v[i]], cand[i]);
            c.low = max(c.low, kFar - (int)cand[i]);
          }
        }
        return;
      }
#pragma unroll
      for (int i = 0; i < E; ++i) {
        go[i] = false;
        if (has[i] && cand[i] < cur[i]) go[i] = cand[i] < umin_atomic(&a.dist[v[i]], cand[i]);
      }
      bool first[E];
      int deg[E];
#pragma unroll
      for (int i = 0; i < E; ++i) {
        first[i] = false;
        if (go[i] && cand[i] < hi) {
          const u64 bit = 1ull << (v[i] & 63);
          u64* w = &next[v[i] >> 6];
          if (!(ld_relaxed(w) & bit)) first[i] = !(atom_or(w, bit) & bit);
        }
      }
#pragma unroll
      for (int i = 0; i < E; ++i) deg[i] = first[i] ? near_degree(a, lite, v[i]) : 0;
#pragma unroll
      for (int i = 0; i < E; ++i) put(first[i], v[i], deg[i], sink, c);
    }
  }

  // Edges of v's row a near round looks at: in a bucket no wider than delta an
  // edge of weight delta or more reaches past it.
  static __device__ __forceinline__ int near_degree(const WArgs& a, bool lite, int v) {
    return lite ? a.light[v] : a.rp[v + 1] - a.rp[v];
  }
  static __device__ __forceinline__ bool lite_rows(const WArgs& a, const State& u) {
    return a.light && uniform(u.width) <= a.delta;
  }

  template <class Sink>
  static __device__ __forceinline__ void put(bool first, int v, int deg, Sink& sink,
                                             SessCount& c) {
    const bool ok = first && deg > 0;
    if (ok) c.mf += (unsigned)deg;
    c.nf += (unsigned)__popcll(__ballot(ok));
    sink.add(ok, v, deg);
  }

  template <int E, class Src, class Sink>
  static __device__ __forceinline__ void push(const WArgs& a, int* own, const State& u,
                                              unsigned phase, unsigned ngroups, unsigned gw, unsigned nwaves,
                                              const Src& src, Sink& sink, SessCount& c) {
    const bool near = phase == kNear;
    const unsigned hi = uniform(u.hi);
    const unsigned par = uniform(u.par);
    u64* mine = par ? a.inq[1] : a.inq[0];
    u64* next = par ? a.inq[0] : a.inq[1];
    const bool split = a.split != 0;
    const bool lite = lite_rows(a, u);
    unsigned du = 0;
    walk_rows<E>(
        own, ngroups, gw, nwaves, src,
        [&](u64 e, unsigned part, int& rs, int& deg) {
          du = 0;
          if (e == kNoEntry) return;
          const int v = (int)(unsigned)e;
          const unsigned piece = (unsigned)(e >> 32);
          rs = a.rp[v];
          deg = near_degree(a, near && lite, v);
          du = (unsigned)ld_relaxed(&a.dist[v]);
          if (near && part == 0 && (piece == 0 || piece == kWhole))
            atomicAnd(&mine[v >> 6], ~(1ull << (v & 63)));
          if (piece != kWhole) {
            rs += (int)piece * kPiece;
            deg = min(kPiece, deg - (int)piece * kPiece);
          }
        },
        [&](const int* o, const int* at, const bool* has0) {
          int v[E];
          unsigned cand[E];
          bool has[E];
#pragma unroll
          for (int q = 0; q < E; ++q) {
            const unsigned d = (unsigned)__shfl((int)du, o[q], kWave);
            cand[q] = has0[q] ? d + (unsigned)a.wt[at[q]] : 0u;
          }
#pragma unroll
          for (int q = 0; q < E; ++q) {
            has[q] = has0[q] && (!split || (cand[q] < hi) == near);
            v[q] = has[q] ? a.col[at[q]] : 0;
          }
          relax<E>(a, near, lite, hi, next, v, cand, has, sink, c);
        });
  }

  // One wave per 64 nodes: rows of the nodes in [lo, hi) to the queue.  settled: they
  // are final; else also the number of nodes less than delta past them and the
  // smallest distance beyond.
  template <class Sink>
  static __device__ __forceinline__ void collect(const WArgs& a, bool settled, bool lite,
                                                 unsigned lo, unsigned hi,
                                                 unsigned gw, unsigned nwaves, Sink& sink,
                                                 SessCount& c) {
    const int lane = lane_id();
    for (unsigned w = gw; w < (unsigned)a.nw; w += 4 * nwaves) {
      unsigned d[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long long v = (long long)(w + q * nwaves) * kWave + lane;
        d[q] = v < a.n ? (unsigned)ld_relaxed(&a.dist[v]) : kUnreached;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int v = (int)((w + q * nwaves) * kWave) + lane;
        const bool in = d[q] >= lo && d[q] < hi;
        if (!settled && d[q] >= hi && d[q] != kUnreached) {
          if (d[q] - hi < a.delta)
            c.scan += 1;
          else
            c.low = max(c.low, kFar - (int)d[q]);
        }
        const u64 bits = __ballot(in);
        if (!bits) continue;
        if (settled && lane == 0) {
          u64* f = &a.fin[w + q * nwaves];
          st_relaxed64(f, ld_relaxed(f) | bits);
        }
        const int deg = in ? near_degree(a, lite && !settled, v) : 0;
        put(in, v, deg, sink, c);
      }
    }
  }

  static __device__ __forceinline__ void wave_low(S& base, const SessCount& c) {
    if (__ballot(c.scan != 0)) return;      // not to be asked for
    const int x = __builtin_amdgcn_readlane(wave_incl_max(c.low), kWave - 1);
    if (lane_id() == 0 && x) atomicMax(&static_cast<Shared&>(base).low, x);
  }

  template <class Sink>
  static __device__ __forceinline__ void step(const WArgs& a, const SessArgs& x, S& sh,
                                              Sink& sink, SessCount& c) {
    const unsigned phase = uniform(sh.p.u.phase);
    level(a, x, sh, phase, sink, c);
    if (phase < kCollect) return;
    wave_low(sh, c);
    __syncthreads();
    const unsigned k = uniform(sh.p.u.lows);
    if (threadIdx.x == 0) {
      Shared& s = static_cast<Shared&>(sh);
      if (s.low)
        __hip_atomic_fetch_max(&a.ctrl->low[k % 3][sh.rank / kSessGroup].v, s.low, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
      s.low = 0;
    }
    // the next such level's words.  They were last read after the one before last, by
    // workgroup 0 and the members of its cluster, which have run a level over all
    // nodes since
    if (sh.rank == 0 && threadIdx.x < kSessGroups)
      st_relaxed(&a.ctrl->low[(k + 1) % 3][threadIdx.x].v, 0);
  }

  template <class Sink>
  static __device__ __forceinline__ void level(const WArgs& a, const SessArgs& x, S& sh,
                                               unsigned phase, Sink& sink, SessCount& c) {
    const int wv = threadIdx.x / kWave;
    const unsigned K = uniform(sh.p.K);
    const unsigned nwaves = K * kSW;
    const unsigned gw = (unsigned)wv * K + sh.rank;
    const State& u = sh.p.u;
    if (uniform(sh.p.scan)) {
      collect(a, phase == kSettled, lite_rows(a, u), uniform(u.lo), uniform(u.hi), gw, nwaves, sink, c);
      return;
    }
    const QueueSrc<WeightPolicy> src = queue_src(sh, x.q[sh.p.qp]);
    const unsigned ngroups = uniform(sh.pre_g[kSessSegs]);
    if (uniform(sh.p.fe) <= nwaves * 2 * kWave)
      push<1>(a, sh.own[wv], u, phase, ngroups, gw, nwaves, src, sink, c);
    else
      push<4>(a, sh.own[wv], u, phase, ngroups, gw, nwaves, src, sink, c);
  }

  template <class Sink>
  static __device__ __forceinline__ void solo(const WArgs& a, S& sh, const u64* cur,
                                              unsigned ncur, Sink& sink, SessCount& c) {
    const int wv = threadIdx.x / kWave;
    const unsigned phase = uniform(sh.p.u.phase);
    push<1>(a, sh.own[wv], sh.p.u, phase, (ncur + kWave - 1) / kWave, (unsigned)wv, (unsigned)kSW,
            ListSrc{cur, ncur}, sink, c);
    if (phase >= kCollect) wave_low(sh, c);
  }

  // What follows the level just run, from the rows it put in the queue (nf, of
  // mf edges), after a collection the nodes less than delta past it, and the smallest
  // distance past the bucket where there is none.
  static __device__ __forceinline__ void advance(const WArgs& a, S& sh, unsigned nf, u64 mf,
                                                 u64 close, bool record) {
    State u = sh.p.u;
    unsigned done = 0;
    u.steps += 1;
    unsigned low = 0;
    if (u.phase >= kCollect) {
      if (sh.p.mode == kModeSolo) {
        low = (unsigned)static_cast<Shared&>(sh).low;
      } else {
        if (!close) {
          const int g = lane_id() & (kSessGroups - 1);
          low = (unsigned)__builtin_amdgcn_readlane(
              wave_incl_max(ld_relaxed(&a.ctrl->low[u.lows % 3][g].v)), kWave - 1);
        }
        u.lows += 1;
      }
    }
    switch (u.phase) {
      case kNear:
        u.rounds += 1;
        u.par ^= 1;
        if (nf) break;
        if (a.split) {
          u.phase = kSettled;
        } else {
          // (no edge is longer than the bucket: the next holds a node, or none is left)
          u.far = (unsigned)kFar - u.hi;
          done = next_bucket(u, a.delta, a.delta);
        }
        break;
      case kSettled:
        // (nobody with an edge: what lies past the bucket is as it was)
        if (nf)
          u.phase = u.gap ? kHeavyGap : kHeavy;
        else
          done = next_bucket(u, a.delta, u.width);
        break;
      case kHeavy:
      case kHeavyGap:
        // (with a gap, the smallest of what lay past it before and what this level made)
        u.far = max(u.far, low);
        // past the bulk of the edges, and on long stretches of next to none, buckets
        // of little work: fewer, wider ones
        u.settled += sh.p.fe;
        u.thin = sh.p.fe <= (unsigned)kSoloCap ? u.thin + 1 : 0;
        done = next_bucket(u, a.delta,
                           (sh.p.fe < kSmallBucket && u.settled > a.half) || u.thin > kThinBuckets
                               ? min(u.width * 2, 1u << 30)
                               : a.delta);
        break;
      default:
        u.gap = close == 0;
        u.far = close ? (unsigned)kFar - u.hi : low;
        if (nf)
          u.phase = kNear;
        else if (a.split)
          u.phase = kSettled;       // its nodes have heavy edges, or none
        else
          done = next_bucket(u, a.delta, u.width);
    }
    if (u.steps > a.max_rounds) done = 2;
    set_plan<WeightPolicy>(sh, done != 0, u.phase == kSettled || u.phase == kCollect, mf, a.nw,
                           kSoloCap);
    if (lane_id() == 0) {
      sh.p.u = u;
      static_cast<Shared&>(sh).low = 0;
      if (done && record) {
        a.ctrl->done = done;
        a.ctrl->rounds = u.rounds;
      }
    }
  }
  // The bucket with the smallest distance left, a whole number of deltas behind this one
  // (R-MAT 20, 8 sources: 7.95 ms, with buckets that start at that distance 8.93: where they
  // begin then depends on the source's lightest edges; width is no less than delta); 1 if there is none.
  static __device__ __forceinline__ unsigned next_bucket(State& u, unsigned delta, unsigned width) {
    if (!u.far) return 1;
    u.phase = kCollect;
    u.lo = u.hi + ((unsigned)kFar - u.far - u.hi) / delta * delta;
    u.width = width;
    u.hi = min(u.lo + width, (unsigned)kFar);
    return 0;
  }

  static __device__ __forceinline__ void begin(const WArgs& a, const SessArgs& x, S& sh) {
    const int s = x.source;
    const int deg = near_degree(a, a.light != nullptr, s);
    if (lane_id() == 0) {
      State& u = sh.p.u;
      u.phase = kCollect;       // as if a collection had found the source
      u.par = 0;
      u.lo = 0;
      u.hi = u.width = a.delta;
      u.rounds = u.steps = u.far = u.gap = u.lows = u.settled = u.thin = 0;
      sh.stage[0] = row_entry(s, deg);
      st_relaxed64(&x.q[0][0], row_entry(s, deg));
    }
    wave_sync();
    advance(a, sh, deg > 0 ? 1u : 0u, (u64)deg, 0ull, true);
  }
};

__global__ __launch_bounds__(kSB, 4) void wsssp_session(WArgs a, SessArgs x) {
  __shared__ WeightPolicy::Shared sh;
  if (threadIdx.x == 0) sh.low = 0;
  session<WeightPolicy>(a, x, sh);
}

// dist = -1 everywhere but the source, bitmaps and control block clear.
__global__ __launch_bounds__(kSB) void wsssp_init(WArgs a, int source) {
  const unsigned tid = blockIdx.x * kSB + threadIdx.x, nt = gridDim.x * kSB;
  if (tid == 0) a.hm->t_start = wall_clock64();
  u64* c = reinterpret_cast<u64*>(a.ctrl);
  for (unsigned i = tid; i < sizeof(WCtrl) / 8; i += nt) c[i] = 0;
  for (unsigned i = tid; i < (unsigned)a.nw; i += nt) {
    a.inq[0][i] = a.inq[1][i] = 0;
    if (a.split) a.fin[i] = 0;
  }
  for (unsigned i = tid; i < (unsigned)a.n; i += nt) a.dist[i] = (int)i == source ? 0 : -1;
}

// A copy of the rows with the edges lighter than delta first (one wave a row).
__global__ __launch_bounds__(kSB) void split_rows(int32_t n, const int32_t* rp, const int32_t* col,
                                                  const int32_t* wt, int32_t delta, int32_t* scol,
                                                  int32_t* swt, int32_t* light) {
  const int lane = lane_id();
  const int nwaves = (int)gridDim.x * kSW;
  for (int v = (int)blockIdx.x * kSW + (int)threadIdx.x / kWave; v < n; v += nwaves) {
    const int s = rp[v], e = rp[v + 1];
    int cnt = 0;
    for (int i = s; i < e; i += kWave)
      cnt += __popcll(__ballot(i + lane < e && wt[i + lane] < delta));
    int nl = s, nh = s + cnt;
    for (int i = s; i < e; i += kWave) {
      const bool in = i + lane < e;
      const int w = in ? wt[i + lane] : 0;
      const u64 lm = __ballot(in && w < delta), hm = __ballot(in && w >= delta);
      if (in) {
        const int at = w < delta ? nl + __popcll(lm & lanes_below()) : nh + __popcll(hm & lanes_below());
        scol[at] = col[i + lane];
        swt[at] = w;
      }
      nl += __popcll(lm);
      nh += __popcll(hm);
    }
    if (lane == 0) light[v] = cnt;
  }
}

// After the run: reached nodes and the sum of their out-degrees (E_reach, the
// GTEPS numerator); the last workgroup reports the end to the host.
__global__ __launch_bounds__(kSB) void wsssp_close(WArgs a) {
  u64 reached = 0, se = 0;
  const int tid = blockIdx.x * kSB + threadIdx.x;
  const int nt = gridDim.x * kSB;
  for (int i = tid; i < a.n; i += nt)
    if (a.dist[i] >= 0) {
      reached += 1;
      se += (u64)(a.rp[i + 1] - a.rp[i]);
    }
  __shared__ u64 red[2][kSW];
  reached = wave_sum(reached);
  se = wave_sum(se);
  if (lane_id() == 0) {
    red[0][threadIdx.x / kWave] = reached;
    red[1][threadIdx.x / kWave] = se;
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  int last = 0;
  if (threadIdx.x == 0) {
    u64 r = 0, e = 0;
    for (int i = 0; i < kSW; ++i) {
      r += red[0][i];
      e += red[1][i];
    }
    WCtrl::Part& p = a.ctrl->part[blockIdx.x % kStripes];
    if (r) {
      atom_add(&p.reached, r);
      atom_add(&p.edges, e);
    }
    wait_all();
    last = atom_add(&a.ctrl->closed, 1u) == gridDim.x - 1;
  }
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  const bool st = lane_id() < kStripes;
  const u64 r = wave_sum(st ? ld_relaxed(&a.ctrl->part[lane_id()].reached) : 0ull);
  const u64 e = wave_sum(st ? ld_relaxed(&a.ctrl->part[lane_id()].edges) : 0ull);
  if (threadIdx.x == 0) {
    a.hm->rounds = a.ctrl->rounds;
    a.hm->done = a.ctrl->done ? a.ctrl->done : 2u;   // 0: a wait timed out
    a.hm->reached = r;
    a.hm->source_edges = e;
    a.hm->t_end = wall_clock64();
    __hip_atomic_store(&a.hm->end_tag, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ------------------------------------------------------------------ host --
namespace {

struct WWs {
  Ctx* ctx = nullptr;
  hipStream_t stream = nullptr;         // of the call that has the workspace
  hipEvent_t ev1 = nullptr;
  u64* q[2] = {nullptr, nullptr};
  u64* inq[2] = {nullptr, nullptr};
  u64* fin = nullptr;
  int32_t* dist = nullptr;
  WCtrl* ctrl = nullptr;
  WMirror* h_m = nullptr;
  WMirror* d_m = nullptr;
  unsigned seq = 0;
  int stripes = kSessStripes;           // sub-queues of the session
  size_t bytes = 0;

  ~WWs() {
    if (stream) hipStreamSynchronize(stream);
    for (int i = 0; i < 2; ++i) {
      dev_free(ctx, q[i], 0);
      dev_free(ctx, inq[i], 0);
    }
    dev_free(ctx, fin, 0);
    dev_free(ctx, dist, 0);
    dev_free(ctx, ctrl, 0);
    if (ctx) ctx->used -= bytes;
    if (h_m) hipHostFree(h_m);
    if (ev1) hipEventDestroy(ev1);
  }
};

dawn_status wws_create(Ctx* ctx, const GraphRec* g, int stripes, std::unique_ptr<WWs>* out) {
  std::unique_ptr<WWs> w(new WWs());
  w->ctx = ctx;
  w->stripes = stripes;
  const size_t n = (size_t)g->n, nw = (n + 63) / 64;
  WWs* wp = w.get();
  auto alloc = [&](void** p, size_t bytes) -> dawn_status {
    dawn_status s = dev_alloc(ctx, p, bytes);
    if (s == DAWN_OK) wp->bytes += bytes;
    return s;
  };
  for (int i = 0; i < 2; ++i) {
    DAWN_TRY(alloc((void**)&w->q[i], (size_t)stripes * sess_queue_cap(g->n, g->m, kWeightPiece) * 8));
    DAWN_TRY(alloc((void**)&w->inq[i], nw * 8));
  }
  DAWN_TRY(alloc((void**)&w->fin, nw * 8));
  DAWN_TRY(alloc((void**)&w->dist, n * 4));
  DAWN_TRY(alloc((void**)&w->ctrl, sizeof(WCtrl)));
  DAWN_HIP(hipHostMalloc((void**)&w->h_m, sizeof(WMirror),
                         hipHostMallocCoherent | hipHostMallocMapped));
  memset(w->h_m, 0, sizeof(WMirror));
  DAWN_HIP(hipHostGetDevicePointer((void**)&w->d_m, w->h_m, 0));
  DAWN_HIP(hipEventCreateWithFlags(&w->ev1, hipEventDisableTiming));
  *out = std::move(w);
  return DAWN_OK;
}

// Spin until run `seq` reports its end, or the work queued before ev1 has all
// run (with or without the report).
hipError_t wait_report(WWs* w, unsigned seq) {
  for (unsigned spin = 1;; ++spin) {
    if (__atomic_load_n(&w->h_m->end_tag, __ATOMIC_ACQUIRE) == seq) return hipSuccess;
    if ((spin & 63) == 0) {
      const hipError_t e = hipEventQuery(w->ev1);
      if (e != hipErrorNotReady) return e;
    }
    __builtin_ia32_pause();
  }
}

}  // namespace

struct WsspPool {
  std::vector<std::unique_ptr<WWs>> ws;
};

void wsssp_pool_free(GraphRec* g) {
  delete reinterpret_cast<WsspPool*>(g->wpool);
  g->wpool = nullptr;
}

LightRows::~LightRows() {
  dev_free(ctx, col, edge_bytes);
  dev_free(ctx, wt, edge_bytes);
  dev_free(ctx, light, node_bytes);
}

Weights::~Weights() { dev_free(ctx, wt, bytes); }

dawn_status wsssp_layout(Ctx* ctx, GraphRec* g, double mean_w, Weights* w) {
  const double mean_deg = std::max((double)g->m / (double)g->n, 1.0);
  double delta = kDelta * mean_w / mean_deg;
  if (delta >= (double)w->max_w) delta = kDeltaWhole * mean_w / mean_deg;
  w->delta = (int32_t)std::min(std::max(delta, 1.0), 1e9);
  if (w->delta >= w->max_w || g->m == 0) return DAWN_OK;
  const size_t mb = (size_t)g->m * 4, nb = (size_t)g->n * 4;
  // only out of plenty
  const uint64_t used = ctx->used.load() + ctx->reserved.load();
  if (used > ctx->budget || 2 * mb + nb > (ctx->budget - used) / 8) return DAWN_OK;
  auto r = std::make_shared<LightRows>();
  r->ctx = ctx;
  r->edge_bytes = mb;
  r->node_bytes = nb;
  if (dev_alloc(ctx, (void**)&r->col, mb) != DAWN_OK ||
      dev_alloc(ctx, (void**)&r->wt, mb) != DAWN_OK ||
      dev_alloc(ctx, (void**)&r->light, nb) != DAWN_OK) {
    // no room for the copy: near rounds then look at whole rows
    clear_error();
    return DAWN_OK;
  }
  hipLaunchKernelGGL(split_rows, dim3(ctx->num_cu * 4), dim3(kSB), 0, 0, g->n, g->rp, g->col, w->wt,
                     w->delta, r->col, r->wt, r->light);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return fail(DAWN_E_DEVICE, "weights layout: %s", hipGetErrorString(e));
  w->rows = std::move(r);
  return DAWN_OK;
}

dawn_status wsssp_run(Ctx* ctx, GraphRec* g, int32_t source, int32_t* dist, bool device_out,
                      dawn_run_stats* stats) {
  const uint64_t t0 = now_ns();
  // (held to the end of the run, which reads them: another call may replace them)
  std::shared_ptr<Weights> weights;
  std::shared_ptr<LightRows> rows;
  std::unique_ptr<WWs> w;
  {
    std::lock_guard<std::mutex> lk(g->mu);
    weights = g->weights;
    if (!weights)
      return fail(DAWN_E_INVALID_ARG, "graph %d has no weights (dawn_graph_set_weights)", g->id);
    WsspPool* pool = reinterpret_cast<WsspPool*>(g->wpool);
    if (pool && !pool->ws.empty()) {
      w = std::move(pool->ws.back());
      pool->ws.pop_back();
    }
  }
  StreamLease lease(ctx);
  DAWN_TRY(lease.take());
  if (!w) {
    dawn_status c = wws_create(ctx, g, kSessStripes, &w);
    // (with one sub-queue, a quarter of the queues' memory: R-MAT 20 x 4 4.59 -> 4.71 ms,
    // grid 1024^2 x 2 3.40 -> 3.78)
    if (c == DAWN_E_NO_MEMORY) c = wws_create(ctx, g, 1, &w);
    DAWN_TRY(c);
  }
  // (a pooled workspace's last launch may still be running)
  else if (w->stream != lease.s) DAWN_HIP(hipStreamWaitEvent(lease.s, w->ev1, 0));
  w->stream = lease.s;
  WArgs a;
  memset(&a, 0, sizeof(a));
  a.n = g->n;
  a.nw = (g->n + 63) / 64;
  a.rp = g->rp;
  a.col = g->col;
  a.dist = device_out ? dist : w->dist;
  a.inq[0] = w->inq[0];
  a.inq[1] = w->inq[1];
  a.ctrl = w->ctrl;
  a.hm = w->d_m;
  w->seq = w->seq % 0x7fffffffu + 1;
  a.seq = w->seq;
  a.fin = w->fin;
  a.half = (unsigned)(g->m / 2);
  {
    std::lock_guard<std::mutex> lk(ctx->rows_mu);
    rows = weights->rows;
  }
  a.wt = weights->wt;
  a.delta = (unsigned)weights->delta;
  a.split = weights->delta < weights->max_w ? 1 : 0;
  if (rows) {
    a.col = rows->col;
    a.wt = rows->wt;
    a.light = rows->light;
  }
  // Every bucket but an empty last one holds a reached node that no earlier one held
  // (distances past a bucket are lowered to no less than its end), so there are at most
  // n + 1.  After
  // r near rounds the nodes are exact whose shortest paths have at most r edges
  // within the bucket, so a bucket of b nodes takes at most b; its collection, that of
  // its settled nodes and the relaxations past it are three levels more.
  a.max_rounds = (unsigned)std::min<long long>(4ll * g->n + 4, 0xffffffffll);
  SessArgs x;
  x.sc = &w->ctrl->sess;
  x.q[0] = w->q[0];
  x.q[1] = w->q[1];
  x.qcap = (unsigned)sess_queue_cap(g->n, g->m, kWeightPiece);
  x.stripes = (unsigned)w->stripes;
  x.ccap = (unsigned)sess_cluster_cap(x.qcap, w->stripes);
  x.source = source;
  hipStream_t s = w->stream;
  const int fill = std::max(1, std::min((g->n + kSB - 1) / kSB, ctx->num_cu * 4));
  static std::atomic<int> occ_cache{0};
  int occ = occ_cache.load(std::memory_order_relaxed);
  hipError_t e = hipSuccess;
  if (!occ) {
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, wsssp_session, kSB, 0);
    occ = std::max(occ, 1);
    if (e == hipSuccess) occ_cache.store(occ, std::memory_order_relaxed);
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(wsssp_init, dim3(fill), dim3(kSB), 0, s, a, source);
    hipLaunchKernelGGL(wsssp_session, dim3(sess_grid(ctx, std::min(occ, kSessPerCu), ctx_share(ctx), a.nw, g->m)),
                       dim3(kSB), 0, s, a, x);
    hipLaunchKernelGGL(wsssp_close, dim3(fill), dim3(kSB), 0, s, a);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipEventRecord(w->ev1, s);
  if (e == hipSuccess) e = wait_report(w.get(), a.seq);
  dawn_status st = DAWN_OK;
  if (e != hipSuccess)
    st = fail(DAWN_E_DEVICE, "weighted SSSP: %s", hipGetErrorString(e));
  else if (w->h_m->end_tag != a.seq || w->h_m->done != 1)
    st = fail(DAWN_E_DEVICE, "weighted level loop did not finish");
  if (st == DAWN_OK && !device_out) {
    e = copy_rows_to_host(ctx, dist, g->n, w->dist, g->n, 1, s);
    if (e != hipSuccess) st = fail(DAWN_E_DEVICE, "weighted SSSP: %s", hipGetErrorString(e));
  }
  if (st != DAWN_OK) return st;   // the workspace is dropped
  const WMirror& m = *w->h_m;
  if (stats) {
    stats->levels = std::max((int32_t)m.rounds, 1);   // rounds that had a frontier
    stats->push_levels = stats->levels;
    stats->pull_levels = 0;
    stats->launches = 3;
    stats->edges_examined = 0;                 // not counted by the weighted rounds
    stats->source_edges = (int64_t)m.source_edges;
    stats->reached = (int64_t)m.reached;
    stats->kernel_ms = ctx->wall_khz > 0 ? (double)(m.t_end - m.t_start) / ctx->wall_khz : 0.0;
    stats->total_ms = (now_ns() - t0) / 1e6;
    stats->kernel_clock_ms = 0.0;
  }
  {
    std::lock_guard<std::mutex> lk(g->mu);
    if (!g->wpool) g->wpool = new WsspPool();
    reinterpret_cast<WsspPool*>(g->wpool)->ws.push_back(std::move(w));
  }
  return DAWN_OK;
}

}  // namespace dawn
