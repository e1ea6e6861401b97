// Batched level loop in one launch, for narrow batches (rows of at most 8
// words: 512 sources).
//
// With few words per node a level of the launch-per-step loop (control, push,
// pull, merge) is mostly launches: on a 512 x 512 grid with 200 sources (four
// words) 20 us of a level's 27 to 95 are spent before and between its kernels,
// and the merge reads again what the expansion wrote.  Here a level is one pass
// over the nodes, and the levels run in one launch (session_dev.hpp):
//
//   new[v]  = act & ~vis[v] & OR over in-neighbours u of vis[u]
//   vis'[v] = vis[v] | new[v]
//
// (the pull step of Algorithm 1 on the visited set, per bit, with its early
// exit), vis and vis' being two buffers used in turn, so that nobody reads a
// bit of the level being run.  A node's row and its level planes are written by
// the lanes that own the node, with no atomics, and there is no frontier to
// keep.  In-lists of at least kPullBig entries are cut into chunks that any
// wave may take; those set their bits with atomic ORs in vis' and the planes:
// vis' still holds the row of two levels ago, a subset, so ORing vis | new in is
// enough, and the old value tells which bits a chunk was first to set.
//
// Early levels meet few visited nodes: a bitmap of the nodes with a nonzero
// row, two buffers likewise, keeps the pass from gathering empty rows until a
// quarter of the nodes is touched.
//
// Measured: 200 sources on the 512 x 512 grid (1 M edges, some 120 levels) 14.7 ms
// before, 2.5 ms now: 15 to 26 us a level, the last ones 11, of which the barrier
// and the reading of the lanes' activity are 5; the rest is the chain in-list ->
// row -> store of the pass, which is why two units go at a time (2.76 ms with
// one).  37 sources on R-MAT of 131 K nodes and 2 M edges: 10 to 42 us a level.
#include <string.h>

#include <algorithm>

#include "batch.hpp"
#include "device_util.hpp"
#include "internal.hpp"
#include "session_dev.hpp"

namespace dawn {

// Edges up to which a level is left to 32 workgroups, whose levels end sooner:
// uniform of 16K nodes and 131K edges, k 64, 153 us against 162 with all; R-MAT of
// 8K and 0.2M edges 200 against 159.
constexpr long long kBsCluster = 128 << 10;
// Edges per node from which lists count as long (launch_t's P): R-MAT of 16K
// nodes and 1.4M edges, k 16, 214 us at one lane a node, 184 at eight.
constexpr long long kBsDense = 24;
constexpr long long kBsEdges = 96ll << 20;
constexpr long long kBsWideEdges = 8ll << 20;
constexpr long long kBsFewEdges = 16ll << 20;

struct BsArgs {
  BatchArgs b;
  FusedCtrl* fc;
};

// Bits 0, P, 2 P, ... of x, side by side.
template <int P>
__device__ __forceinline__ u64 compress(u64 x) {
  if constexpr (P == 2) {
    x = (x | x >> 1) & 0x3333333333333333ull;
    x = (x | x >> 2) & 0x0f0f0f0f0f0f0f0full;
    x = (x | x >> 4) & 0x00ff00ff00ff00ffull;
    x = (x | x >> 8) & 0x0000ffff0000ffffull;
    x = (x | x >> 16) & 0x00000000ffffffffull;
  } else if constexpr (P == 4) {
    x = (x | x >> 3) & 0x0303030303030303ull;
    x = (x | x >> 6) & 0x000f000f000f000full;
    x = (x | x >> 12) & 0x000000ff000000ffull;
    x = (x | x >> 24) & 0x000000000000ffffull;
  } else if constexpr (P == 8) {
    x = (x | x >> 7) & 0x0003000300030003ull;
    x = (x | x >> 14) & 0x0000000f0000000full;
    x = (x | x >> 28) & 0x00000000000000ffull;
  }
  return x;
}

template <int P>
struct BatchPolicy {
  static constexpr int kPiece = 64;
  // (the planes are read and written by their nodes' owner at every level)
  static constexpr bool kAdmits = false;
  template <class Plan>
  static __device__ __forceinline__ unsigned long long join_ticks(const Plan&, int) {
    return kJoinLong;
  }
  using Args = BsArgs;
  struct State {
    unsigned level;             // being run
    unsigned buf;               // vis buffer that holds the levels before it
    unsigned touched;           // nodes with a nonzero row
    unsigned last;              // last level that found something
  };
  struct Shared : SessShared<BatchPolicy> {
    u64 act[8];                 // sources that found something at the last level
    u64 found[8];               // ... at this one
    u64 edges, reached, degs;   // this workgroup's totals over the levels
  };
  using S = SessShared<BatchPolicy>;

  static __device__ __forceinline__ u64 entry(int, int, int) { return 0; }
  static __device__ __forceinline__ u64 row_entry(int, int) { return 0; }
  // Units of a level's pass (P to a word) and chunks, a wave each.  With more
  // than kBsCluster edges 32 workgroups are too few.
  static __device__ __forceinline__ int words(const BsArgs& a) {
    const int x = (a.b.n + 63) / 64 * P + a.b.npc;
    return a.b.m > kBsCluster ? max(x, kClusterWords + 1) : x;
  }
  static __device__ __forceinline__ bool scans(const SessPlan<State>&) { return true; }
  template <class Sink>
  static __device__ __forceinline__ void solo(const BsArgs&, S&, const u64*, unsigned, Sink&,
                                              SessCount&) {}

  // In-edges [s, e) scanned by the whole wave, 64 a step; needw / accw: needed
  // and found bits per word, wave-uniform.
  static __device__ __forceinline__ unsigned wave_rows(const BatchArgs& b, const u64* vis,
                                                       const u64* any, bool sparse, int s, int e,
                                                       const u64* needw, u64* accw) {
    const int lane = lane_id();
    int j = s;
    while (j < e) {
      u64 row[P];
#pragma unroll
      for (int x = 0; x < P; ++x) row[x] = 0;
      if (j + lane < e) {
        const int u = b.isrc[j + lane];
        if (!sparse || ((ld_relaxed(&any[u >> 6]) >> (u & 63)) & 1ull)) {
          const u64* r = vis + (size_t)u * (size_t)b.Ws;
#pragma unroll
          for (int x = 0; x < P; ++x)
            if (x < b.W) row[x] = ld_relaxed(r + x) & needw[x];
        }
      }
      j += kWave;
      bool done = true;
#pragma unroll
      for (int x = 0; x < P; ++x) {
        if (__ballot((row[x] & ~accw[x]) != 0)) accw[x] |= wave_or(row[x]);
        done = done && accw[x] == needw[x];
      }
      if (done) break;
    }
    return (unsigned)(min(j, e) - s);
  }

  // Planes read ahead per unit (a level's number seldom has more bits set).
  static constexpr int kEarly = 3;

  template <class Sink>
  static __device__ __forceinline__ void step(const BsArgs& a, const SessArgs&, S& base, Sink&,
                                              SessCount& c) {
    Shared& sh = static_cast<Shared&>(base);
    const BatchArgs& b = a.b;
    const int t = threadIdx.x, wv = t / kWave, lane = lane_id();
    const State& u = sh.p.u;
    const unsigned L = uniform(u.level);
    const bool second = uniform(u.buf) != 0;
    const u64* vis = second ? b.nxt[0] : b.vis;
    u64* out = second ? b.vis : b.nxt[0];
    const u64* any = second ? b.touched[1] : b.touched[0];
    u64* any_out = second ? b.touched[0] : b.touched[1];
    const bool sparse = uniform(u.touched) < (unsigned)b.n / 4;
    const size_t W = (size_t)b.Ws;
    // who is still expanding
    if (t < 8) sh.act[t] = sh.found[t] = 0;
    __syncthreads();
    if (t < kStripes * 8) {
      const u64 x = (t & 7) < b.W ? ld_relaxed(&a.fc->lact[(L - 1) % 3][t >> 3].w[t & 7]) : 0ull;
      if (x) atomicOr(&sh.act[t & 7], x);
    }
    if (sh.rank == 0 && t < kStripes * 8)
      st_relaxed64(&a.fc->lact[(L + 1) % 3][t >> 3].w[t & 7], 0ull);
    __syncthreads();
    const unsigned nwaves = uniform(sh.p.K) * kSW;
    const unsigned gw = (unsigned)wv * uniform(sh.p.K) + sh.rank;
    u64 edges = 0, reached = 0, degs = 0;
    u64 act_all[P];
#pragma unroll
    for (int x = 0; x < P; ++x) act_all[x] = sh.act[x];

    // long in-lists, a wave per chunk
    for (unsigned ch = gw; ch < (unsigned)b.npc; ch += nwaves) {
      const int v = b.pcv[ch];
      const int s = b.ip[v] + b.pck[ch] * kPullChunk;
      const int e = min(s + kPullChunk, b.ip[v + 1]);
      const u64 mine = lane < b.W ? ld_relaxed(&vis[(size_t)v * W + lane]) : 0ull;
      u64 needw[P], accw[P];
      bool want = false;
#pragma unroll
      for (int x = 0; x < P; ++x) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mine, x);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mine >> 32), x);
        needw[x] = x < b.W ? act_all[x] & ~(((u64)hi << 32) | lo) : 0ull;
        accw[x] = 0;
        want = want || needw[x] != 0;
      }
      if (want) {
        const unsigned nr = wave_rows(b, vis, any, sparse, s, e, needw, accw);
        if (lane == 0) edges += nr;
      }
      u64 got = 0;
      bool hit = false;
#pragma unroll
      for (int x = 0; x < P; ++x) {
        if (x == lane) got = accw[x];
        hit = hit || accw[x] != 0;
      }
      if (lane < b.W && (mine | got)) {
        const size_t idx = (size_t)v * W + lane;
        // the first chunk to set a bit counts it
        const u64 fresh = got & ~atom_or(&out[idx], mine | got);
        for (unsigned r = fresh ? L : 0u; r; r &= r - 1) atom_or(&b.planes[__builtin_ctz(r)][idx], fresh);
        if (fresh) {
          const u64 k = (u64)__popcll(fresh);
          reached += k;
          degs += k * (u64)(b.rp[v + 1] - b.rp[v]);
          atomicOr(&sh.found[lane], fresh);
        }
      }
      if (hit) c.nf += 1;
      const bool was = __ballot(mine != 0) != 0;
      if (lane == 0 && (was || hit)) {
        const u64 bit = 1ull << (v & 63);
        const u64 old = atom_or(&any_out[v >> 6], bit);
        if (!was && !(old & bit)) c.scan += 1;
      }
    }

    // the planes that take this level's bits: the first few by register
    int plane[kEarly];
    unsigned rest = L & ((1u << b.nplanes) - 1u);
#pragma unroll
    for (int m = 0; m < kEarly; ++m) {
      plane[m] = rest ? __builtin_ctz(rest) : -1;
      rest &= rest - 1;
    }

    // the other nodes: a wave per 64 / P of them, a group of P lanes per node
    constexpr int NPW = kWave / P;
    const int w = lane & (P - 1), sub = lane / P;
    const bool wok = w < b.W;
    const u64 gm = P == 1 ? 1ull << lane : ((1ull << P) - 1ull) << (lane & ~(P - 1));
    const u64 actw = wok ? sh.act[w] : 0ull;
    u64 found = 0;
    const unsigned units = (unsigned)((b.n + 63) / 64) * P;
    // U units at a time, their loads in flight together
    constexpr int U = P <= 4 ? 2 : 1;
    for (unsigned un = gw; un < units; un += U * nwaves) {
      int v[U], s[U], e[U], j[U];
      bool valid[U], big[U], wide[U], go[U];
      u64 vw[U], need[U], gneed[U], acc[U], pl[U][kEarly];
      bool any_go = false;
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const unsigned x = un + (unsigned)k * nwaves;
        v[k] = (int)(x / P) * 64 + (int)(x % P) * NPW + sub;
        valid[k] = x < units && v[k] < b.n;
        s[k] = e[k] = 0;
        vw[k] = 0;
        if (valid[k]) {
          s[k] = b.ip[v[k]];
          e[k] = b.ip[v[k] + 1];
          if (wok) vw[k] = ld_relaxed(&vis[(size_t)v[k] * W + w]);
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        big[k] = e[k] - s[k] >= kPullBig;      // went by chunks
        need[k] = valid[k] && !big[k] ? actw & ~vw[k] : 0ull;
        gneed[k] = __ballot(need[k] != 0) & gm;
        wide[k] = e[k] - s[k] > b.wide_scan;
        acc[k] = 0;
        j[k] = s[k];
        go[k] = gneed[k] != 0 && !wide[k] && !big[k] && s[k] < e[k];
        any_go = any_go || go[k];
        // the planes' words, read while the search is under way
#pragma unroll
        for (int m = 0; m < kEarly; ++m)
          pl[k][m] = need[k] && plane[m] >= 0 ? b.planes[plane[m]][(size_t)v[k] * W + w] : 0ull;
      }
      while (__ballot(any_go)) {
        int uu[U][4];
        u64 val[U][4];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            uu[k][q] = go[k] && j[k] + q < e[k] ? b.isrc[j[k] + q] : -1;
        if (sparse) {
#pragma unroll
          for (int k = 0; k < U; ++k) {
            u64 an[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
              an[q] = uu[k][q] >= 0 ? ld_relaxed(&any[uu[k][q] >> 6]) : 0ull;
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (uu[k][q] >= 0 && !((an[q] >> (uu[k][q] & 63)) & 1ull)) uu[k][q] = -1;
          }
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            val[k][q] = uu[k][q] >= 0 && wok ? ld_relaxed(&vis[(size_t)uu[k][q] * W + w]) : 0ull;
        any_go = false;
#pragma unroll
        for (int k = 0; k < U; ++k) {
          acc[k] |= (val[k][0] | val[k][1] | val[k][2] | val[k][3]) & need[k];
          if (go[k]) {
            if (w == 0) edges += (u64)min(4, e[k] - j[k]);
            j[k] += 4;
          }
          const bool more = (__ballot(acc[k] != need[k]) & gm) != 0;
          go[k] = go[k] && more && j[k] < e[k];
          any_go = any_go || go[k];
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        // lists longer than wide_scan: the whole wave
        u64 lead = __ballot(wide[k] && !big[k] && gneed[k] != 0 && w == 0);
        while (lead) {
          const int ld = __ffsll((unsigned long long)lead) - 1;
          lead &= lead - 1;
          const int ss = __builtin_amdgcn_readlane(s[k], ld);
          const int ee = __builtin_amdgcn_readlane(e[k], ld);
          u64 needw[P], accw[P];
#pragma unroll
          for (int x = 0; x < P; ++x) {
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)need[k], ld + x);
            const unsigned hi =
                (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(need[k] >> 32), ld + x);
            needw[x] = ((u64)hi << 32) | lo;
            accw[x] = 0;
          }
          const unsigned nr = wave_rows(b, vis, any, sparse, ss, ee, needw, accw);
          if (lane == 0) edges += nr;
#pragma unroll
          for (int x = 0; x < P; ++x)
            if (lane == ld + x) acc[k] = accw[x];
        }
        const unsigned x = un + (unsigned)k * nwaves;
        if (valid[k] && wok && !big[k]) {
          const size_t idx = (size_t)v[k] * W + w;
          st_relaxed64(&out[idx], vw[k] | acc[k]);
          if (acc[k]) {
#pragma unroll
            for (int m = 0; m < kEarly; ++m)
              if (plane[m] >= 0) b.planes[plane[m]][idx] = pl[k][m] | acc[k];
            for (unsigned r = rest; r; r &= r - 1) b.planes[__builtin_ctz(r)][idx] |= acc[k];
            const u64 cnt = (u64)__popcll(acc[k]);
            reached += cnt;
            degs += cnt * (u64)(b.rp[v[k] + 1] - b.rp[v[k]]);
            found |= acc[k];
          }
        }
        const u64 hit = __ballot(acc[k] != 0);
        c.nf += hit != 0 ? 1u : 0u;
        // a bit per node: has it a row now, had it one before
        const u64 zw = __ballot(!big[k] && vw[k] != 0);
        const u64 za = __ballot(!big[k] && (vw[k] | acc[k]) != 0);
        const u64 was = compress<P>(__ballot(w == 0 && (zw & gm) != 0));
        const u64 nz = compress<P>(__ballot(w == 0 && (za & gm) != 0));
        if (lane == 0 && nz) {
          // (long lists' nodes add their own bits)
          atom_or(&any_out[x / P], nz << ((x % P) * NPW));
          c.scan += (unsigned)__popcll(nz & ~was);
        }
      }
    }
    // lanes w, w + P, ... hold the same word
    if (found && wok) atomicOr(&sh.found[w], found);
    edges = wave_sum(edges);
    reached = wave_sum(reached);
    degs = wave_sum(degs);
    if (lane == 0 && (edges | reached)) {
      atomicAdd(&sh.edges, edges);
      atomicAdd(&sh.reached, reached);
      atomicAdd(&sh.degs, degs);
    }
    __syncthreads();
    if (t < b.W && sh.found[t])
      atom_or(&a.fc->lact[L % 3][sh.rank % kStripes].w[t], sh.found[t]);
  }

  // The level found something or the run ends; a level past the planes waits
  // for more of them (done = 4).
  static __device__ __forceinline__ void advance(const BsArgs& a, S& sh, unsigned nf, u64,
                                                 u64 touched, bool record_) {
    State u = sh.p.u;
    const unsigned L = u.level;
    int done = 0;
    if (nf) u.last = L;
    u.touched += (unsigned)touched;
    u.buf ^= 1;
    u.level = L + 1;
    if (!nf)
      done = 1;
    else
      done = stop(a, L + 1);
    set_plan<BatchPolicy>(sh, done != 0, true, 0ull, words(a), 0);
    if (lane_id() == 0) {
      sh.p.u = u;
      if (done && record_) leave(a, u, done);
    }
  }
  static __device__ __forceinline__ int stop(const BsArgs& a, unsigned L) {
    if (L > (unsigned)a.b.n + 1u) return 2;
    return 32 - __clz((int)L) > a.b.nplanes ? 4 : 0;
  }
  static __device__ __forceinline__ void leave(const BsArgs& a, const State& u, int done) {
    BatchRun* r = &a.b.ctrl->run;
    r->done = done;
    r->last_nonempty = (int)u.last;
    r->pull_levels = (int)u.level - 1;
    r->vis_buf = (int)u.buf;
    a.fc->level = u.level;
    a.fc->touched = u.touched;
    if (done == 2) atomicMax(&a.b.flags[kFlagStatus], 2u);
  }

  static __device__ __forceinline__ void begin(const BsArgs& a, const SessArgs&, S& sh) {
    BatchRun* r = &a.b.ctrl->run;
    const unsigned bad = ld_relaxed(&a.b.flags[kFlagStatus]);
    State u;
    u.level = a.fc->level;
    u.buf = (unsigned)r->vis_buf;
    u.touched = a.fc->touched;
    u.last = (unsigned)r->last_nonempty;
    const int done = r->done == 1 ? 1 : bad ? 3 : stop(a, u.level);
    if (lane_id() == 0) sh.p.u = u;
    wave_sync();
    set_plan<BatchPolicy>(sh, done != 0, true, 0ull, words(a), 0);
    if (lane_id() == 0 && done != 1) {
      // (a run that goes on after a stop for planes still says so: one that ends without
      // a word of its own must not be taken for stopped again)
      if (done)
        leave(a, u, done);
      else
        r->done = 0;
    }
  }
};

template <int P>
__global__ __launch_bounds__(kSB, 4) void batch_session(BsArgs a, SessArgs x) {
  __shared__ typename BatchPolicy<P>::Shared sh;
  if (threadIdx.x == 0) sh.edges = sh.reached = sh.degs = 0;
  session<BatchPolicy<P>>(a, x, sh);
  if (threadIdx.x == 0 && (sh.edges | sh.reached)) {
    FusedPart& p = a.fc->part[blockIdx.x % kStripes];
    atom_add(&p.edges, sh.edges);
    atom_add(&p.reached, sh.reached);
    atom_add(&p.degs, sh.degs);
  }
}

// Level 0: source i's bit in its row, both bitmaps of touched nodes, the
// totals.  A source outside [0, n) is skipped (device-ordered calls find it
// beforehand and stop the run).
__global__ __launch_bounds__(256) void batch_session_seed(BsArgs a, const int32_t* src, int k) {
  const BatchArgs& b = a.b;
  if (blockIdx.x == 0 && threadIdx.x == 0) b.flags[kFlagDirty] = 1;
  const int i = (int)(blockIdx.x * 256 + threadIdx.x);
  u64 reached = 0, degs = 0, touched = 0;
  if (i < k && (unsigned)src[i] < (unsigned)b.n) {
    const int s = src[i];
    atom_or(&b.vis[(size_t)s * (size_t)b.Ws + (i >> 6)], 1ull << (i & 63));
    const u64 bit = 1ull << (s & 63);
    touched = (atom_or(&b.touched[0][s >> 6], bit) & bit) ? 0 : 1;
    atom_or(&a.fc->lact[0][blockIdx.x % kStripes].w[i >> 6], 1ull << (i & 63));
    reached = 1;
    degs = (u64)(b.rp[s + 1] - b.rp[s]);
  }
  reached = wave_sum(reached);
  degs = wave_sum(degs);
  const unsigned nt = wave_sum((unsigned)touched);
  if (lane_id() == 0) {
    FusedPart& p = a.fc->part[blockIdx.x % kStripes];
    atom_add(&p.reached, reached);
    atom_add(&p.degs, degs);
    atom_add(&a.fc->touched, nt);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.fc->level = 1;
  }
}

// ------------------------------------------------------------------ host --
// Where a run of k sources (W words) takes this path.  The pass reads all rows
// and in-lists of the nodes still wanted; the launch-per-step loop can push the
// first levels from a few nodes instead.  Measured, this path / that one, us:
//  * R-MAT of 8K nodes and 0.2M edges, k 64: 159 / 406; of 131K and 1.9M: 208 /
//    386; of 262K and 7.6M: 341 / 572; of 1M and 31M: 1144 / 1941; uniform of 1M
//    and 12.6M: 984 / 1986.  The gain ends with the caches: R-MAT of 4M nodes and
//    128M edges 8250 / 7582.
//  * rows of five to eight words are whole lines, which the pushes then use as
//    well as the pulls do: k 512 on R-MAT of 262K and 7.6M 1141 / 1272, of 131K
//    and 7.1M 903 / 915, but of 262K and 14.5M 1556 / 1447, of 1M and 31M 4335 /
//    3786; with few edges to a node it wins at any size (uniform of 4M nodes
//    and 67M edges 12283 / 16101, R-MAT of 524K and 8M 1692 / 2068).
//  * few sources leave most of a large graph's first levels empty: k 1 on R-MAT
//    of 262K and 14.5M 330 / 354, of 131K and 19.3M 385 / 330, of 2M and 64M 1750 /
//    1232; k 16 there 2234 / 2993.
bool batch_session_fits(const GraphRec* g, const dawn_params& p, int k) {
  const int W = (k + 63) / 64;
  if (W > 8 || p.direction == 1 || g->m > kBsEdges) return false;
  if (W > 4 && g->m > std::max(kBsWideEdges, 20ll * g->n)) return false;
  return k >= 16 || g->m <= kBsFewEdges;
}

dawn_status batch_session_seed_launch(const BatchArgs& a, FusedCtrl* fc, const int32_t* d_src,
                                      int k, hipStream_t s) {
  BsArgs x{a, fc};
  hipLaunchKernelGGL(batch_session_seed, dim3((k + 255) / 256), dim3(256), 0, s, x, d_src, k);
  DAWN_HIP(hipGetLastError());
  return DAWN_OK;
}

template <int P>
static dawn_status launch_t(Ctx* ctx, const BatchArgs& a, FusedCtrl* fc, hipStream_t s) {
  static std::atomic<int> occ_cache{0};
  int occ = occ_cache.load(std::memory_order_relaxed);
  if (!occ) {
    DAWN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, batch_session<P>, kSB, 0));
    occ = std::max(occ, 1);
    occ_cache.store(occ, std::memory_order_relaxed);
  }
  BsArgs b{a, fc};
  SessArgs x;
  memset(&x, 0, sizeof(x));
  x.sc = &fc->sess;
  x.stripes = 1;
  const int grid = sess_grid(ctx, std::min(occ, kSessPerCu), ctx_share(ctx, false),
                             std::max((a.n + 63) / 64 * P + a.npc, kSessGroup * kSW), 0);
  hipLaunchKernelGGL(batch_session<P>, dim3(grid), dim3(kSB), 0, s, b, x);
  DAWN_HIP(hipGetLastError());
  return DAWN_OK;
}

dawn_status batch_session_launch(Ctx* ctx, const BatchArgs& a, FusedCtrl* fc, hipStream_t s) {
  // a group of P lanes per node; more lanes than words where the lists are long
  // and the nodes few, since a wave scans its longer lists one after another
  int P = a.W <= 1 ? 1 : a.W <= 2 ? 2 : a.W <= 4 ? 4 : 8;
  while (P < 8 && a.m > kBsDense * (long long)a.n && (a.n + 63) / 64 * P < ctx->num_cu * kSW) P *= 2;
  if (a.W <= P) {
    if (P == 1) return launch_t<1>(ctx, a, fc, s);
    if (P == 2) return launch_t<2>(ctx, a, fc, s);
    if (P == 4) return launch_t<4>(ctx, a, fc, s);
    return launch_t<8>(ctx, a, fc, s);
  }
  return fail(DAWN_E_INVALID_ARG, "batch too wide for a session");
}

}  // namespace dawn
