// The session frame and its policies on the host, under random schedules:
// session_emu hop|weighted|batch SEED0 SEEDS [grid=N hold=P held=N late=P ...].
// join: every workgroup has to be a member in the end.
// Prints one line and exits nonzero at the first run whose distances or totals
// differ from a plain search's.
#include <hip/hip_runtime.h>

#include <stdio.h>

#include <queue>
#include <random>

#include "bsession.hip"
#include "session.hip"
#include "wsssp.hip"

#include "emu.hpp"

namespace dawn {
dawn_status fail(dawn_status st, const char*, ...) { return st; }
void clear_error() {}
dawn_status dev_alloc(Ctx*, void**, size_t, bool) { return DAWN_E_NO_MEMORY; }
void dev_free(Ctx*, void*, size_t) {}
hipError_t copy_rows_to_host(Ctx*, int32_t*, size_t, const int32_t*, size_t, size_t, hipStream_t) {
  return hipSuccess;
}
}  // namespace dawn
namespace dawn {
dawn_status StreamLease::take() { return DAWN_OK; }
StreamLease::~StreamLease() {}
}  // namespace dawn
using namespace dawn;

struct Graph {
  int n = 0;
  std::vector<int> rp, col, ip, isrc, wt;
  std::vector<u64> noin;
};

// Stretches of one node a level, fans of up to `wide` nodes, random edges between
// near levels: frontiers of one edge up to a few hundred, in no order; first a path.
static Graph make(std::mt19937_64& g, int levels, int wide, int wmax, int path) {
  std::vector<std::vector<int>> at(levels);
  int n = 0;
  int width = 1;
  for (int l = 0; l < levels; ++l) {
    if (l < path) width = 1;
    else if (g() % 5 == 0) width = 1 + (int)(g() % (unsigned)wide);
    else if (g() % 3 == 0) width = 1;
    for (int i = 0; i < width; ++i) at[l].push_back(n++);
  }
  n += 3;                                  // and some no path leads to
  std::vector<std::pair<int, int>> e;
  for (int l = 1; l < levels; ++l)
    for (int v : at[l]) {
      e.push_back({at[l - 1][g() % at[l - 1].size()], v});
      for (int k = (int)(g() % 4); k > 0; --k) {
        const int a = std::max(0, l - 1 - (int)(g() % 3));
        e.push_back({at[a][g() % at[a].size()], v});
        if (g() % 2) e.push_back({v, at[a][g() % at[a].size()]});
      }
    }
  std::sort(e.begin(), e.end());
  Graph r;
  r.n = n;
  r.rp.assign(n + 1, 0);
  r.ip.assign(n + 1, 0);
  for (auto& x : e) ++r.rp[x.first + 1], ++r.ip[x.second + 1];
  for (int i = 0; i < n; ++i) r.rp[i + 1] += r.rp[i], r.ip[i + 1] += r.ip[i];
  r.isrc.resize(e.size() + 1);
  std::vector<int> pos(r.ip.begin(), r.ip.end() - 1);
  for (auto& x : e) {
    r.col.push_back(x.second);
    r.wt.push_back(g() % 8 ? (int)(g() % 3) : (int)(g() % (unsigned)wmax));
    r.isrc[pos[x.second]++] = x.first;
  }
  r.col.push_back(0);
  r.wt.push_back(0);
  r.noin.assign((n + 63) / 64, 0);
  for (int v = 0; v < n; ++v)
    if (r.ip[v] == r.ip[v + 1]) r.noin[v / 64] |= 1ull << (v % 64);
  return r;
}

static std::vector<int> search(const Graph& g, int s, bool weighted) {
  std::vector<int> d(g.n, -1);
  std::priority_queue<std::pair<int, int>> q;
  q.push({0, s});
  while (!q.empty()) {
    const int du = -q.top().first, u = q.top().second;
    q.pop();
    if (d[u] >= 0) continue;
    d[u] = du;
    for (int i = g.rp[u]; i < g.rp[u + 1]; ++i)
      if (d[g.col[i]] < 0) q.push({-(du + (weighted ? g.wt[i] : 1)), g.col[i]});
  }
  return d;
}

struct Queues {
  std::vector<u64> q[2];
  SessArgs x{};
  Queues(const Graph& g, int piece, SessCtrl* sc, int s, int stripes) {
    x.qcap = (unsigned)sess_queue_cap(g.n, (long long)g.col.size() - 1, piece);
    x.stripes = (unsigned)stripes;
    x.ccap = (unsigned)sess_cluster_cap(x.qcap, stripes);
    x.sc = sc;
    x.source = s;
    for (int i = 0; i < 2; ++i) {
      q[i].assign((size_t)stripes * x.qcap, ~0ull - 5);     // (no entry stands for a row)
      x.q[i] = q[i].data();
    }
  }
};

// Members of the last record.
template <class P>
static unsigned members(const SessCtrl& sc) {
  return (unsigned)sc.rec[offsetof(SessPlan<typename P::State>, members) / 4];
}

static int failed(const char* what, unsigned long long seed) {
  printf("seed %llu: %s\n", seed, what);
  return 1;
}

// A narrow batch of k sources on P words, its level planes growing by one from run to
// run.  stall: the second run's barrier is made to time out, and that run has to
// be told from one that wants more planes (it has enough of them).
template <int P>
static const char* batch(const Graph& g, int k, emu::Launch l, bool stall) {
  const int nw = (g.n + 63) / 64;
  std::unique_ptr<BatchCtrl> ctrl(new BatchCtrl());
  std::unique_ptr<FusedCtrl> fc(new FusedCtrl());
  memset((void*)ctrl.get(), 0, sizeof(BatchCtrl));
  memset((void*)fc.get(), 0, sizeof(FusedCtrl));
  std::vector<u64> vis((size_t)g.n * P, 0), nxt(vis), t0(nw, 0), t1(nw, 0);
  std::vector<std::vector<u64>> planes;
  unsigned flags[2] = {1, 0};
  std::vector<int> pcv, pck;
  for (int v = 0; v < g.n; ++v)
    if (g.ip[v + 1] - g.ip[v] >= kPullBig)
      for (int i = 0; i * kPullChunk < g.ip[v + 1] - g.ip[v]; ++i) pcv.push_back(v), pck.push_back(i);
  BsArgs a;
  memset((void*)&a, 0, sizeof(a));
  a.fc = fc.get();
  BatchArgs& b = a.b;
  b.n = g.n, b.W = b.Ws = (k + 63) / 64, b.m = (long long)g.col.size() - 1;
  b.rp = g.rp.data(), b.col = g.col.data(), b.ip = g.ip.data(), b.isrc = g.isrc.data();
  b.pcv = pcv.data(), b.pck = pck.data(), b.npc = (int)pcv.size();
  b.vis = vis.data(), b.nxt[0] = nxt.data();
  b.touched[0] = t0.data(), b.touched[1] = t1.data();
  b.ctrl = ctrl.get(), b.flags = flags, b.wide_scan = 8;
  std::vector<int> src(k);
  for (int i = 0; i < k; ++i) {
    const int s = src[i] = i == 0 ? 0 : (int)((unsigned)i * 2654435761u % (unsigned)g.n);
    vis[(size_t)s * b.Ws + i / 64] |= 1ull << (i % 64);
    if (!((t0[s / 64] >> (s % 64)) & 1)) ++fc->touched;
    t0[s / 64] |= 1ull << (s % 64);
    fc->lact[0][0].w[i / 64] |= 1ull << (i % 64);
    ++fc->part[0].reached;
  }
  fc->level = 1;
  SessArgs x;
  memset((void*)&x, 0, sizeof(x));
  x.sc = &fc->sess;
  x.stripes = 1;
  for (int run = 0;; ++run) {
    for (int i = 0; i < (stall && run == 1 ? 4 : 1); ++i) planes.emplace_back(vis.size(), 0ull);
    b.nplanes = (int)planes.size();
    for (int i = 0; i < b.nplanes; ++i) b.planes[i] = planes[i].data();
    if (run) memset((void*)&fc->sess, 0, sizeof(SessCtrl));
    l.stalled = stall && run == 1 ? (int)l.grid / 2 : -1;
    std::vector<std::unique_ptr<typename BatchPolicy<P>::Shared>> sh(l.grid);
    for (auto& p : sh) p.reset(new typename BatchPolicy<P>::Shared()), p->edges = p->reached = p->degs = 0;
    if (!emu::run(l, [&](unsigned w) { session<BatchPolicy<P>>(a, x, *sh[w]); })) return "no end";
    for (auto& p : sh) fc->part[0].reached += p->reached;
    if (l.stalled >= 0) return ctrl->run.done == 0 ? nullptr : "a run that timed out says otherwise";
    if (ctrl->run.done != 4) break;
  }
  if (ctrl->run.done != 1) return "not done";
  const std::vector<u64>& rows = ctrl->run.vis_buf ? nxt : vis;
  u64 reached = 0;
  for (int i = 0; i < k; ++i) {
    const std::vector<int> want = search(g, src[i], false);
    for (int v = 0; v < g.n; ++v) {
      const size_t at = (size_t)v * b.Ws + i / 64;
      int d = -1;
      if ((rows[at] >> (i % 64)) & 1) {
        d = 0;
        for (int p = 0; p < b.nplanes; ++p) d |= (int)((planes[p][at] >> (i % 64)) & 1) << p;
        ++reached;
      }
      if (d != want[v]) return "distances";
    }
  }
  return reached == fc->part[0].reached ? nullptr : "totals";
}

// A row of nearly 2^31 edges, as the last wave of the largest launch walks it.
static const char* walk() {
  const int start = 7, deg = 0x7fffffff - 64;
  unsigned long long seen = 0, mine = 0;
  bool out = false;
  std::vector<int> own(4 * kWave);
  const unsigned nwaves = kSessGroups * kSessGroup * 8;
  struct {
    u64 get(unsigned, int lane) const { return lane ? kNoEntry : 1ull; }
  } src;
  emu::Launch l;
  l.grid = 1;
  l.block = 64;
  l.limit = 1000000;
  const unsigned long long used = emu::run(l, [&](unsigned) {
    walk_rows<4>(
        own.data(), 1, nwaves - 1, nwaves, src,
        [&](u64 e, unsigned, int& rs, int& d) {
          if (e == kNoEntry) return;
          rs = start;
          d = deg;
        },
        [&](const int* o, const int* at, const bool* has) {
          for (int q = 0; q < 4; ++q)
            if (has[q]) {
              ++seen;
              out = out || o[q] != 0 || at[q] < start || at[q] - start >= deg;
            }
        });
  });
  const unsigned long long step = 2ull * nwaves * 256;       // two shares a wave
  for (unsigned long long part : {(unsigned long long)nwaves - 1, 2ull * nwaves - 1})
    for (unsigned long long e = part * 256; e < (unsigned long long)deg; e += step)
      mine += std::min<unsigned long long>(256, (unsigned long long)deg - e);
  if (!used) return "no end";
  if (out) return "an edge outside the row";
  return seen == mine ? nullptr : "edges";
}

// The part of the device that a call's session may take.
static const char* callers() {
  Ctx c;
  auto pause = [](int ms) { std::this_thread::sleep_for(std::chrono::milliseconds(ms)); };
  if (ctx_share(&c) != 1) return "idle";
  {
    Caller one(&c);
    if (ctx_share(&c) != 1) return "one caller";
  }
  for (int i = 0; i < 3; ++i) {
    Caller one(&c);
    if (ctx_share(&c) != 1) return "one caller, again and again";
  }
  {
    Caller one(&c), two(&c);
    if (ctx_share(&c) != 2) return "two callers";
    Caller three(&c), four(&c), five(&c);
    if (ctx_share(&c) != kMaxShare) return "five callers";
  }
  if (ctx_share(&c) != kMaxShare) return "just after";
  pause(5);
  {
    Caller one(&c);
    if (ctx_share(&c) != 1) return "later";
    c.queued_ns = now_ns();
    if (ctx_share(&c) != 2 || ctx_share(&c, false) != 1) return "beside queued work";
  }
  pause(5);
  return ctx_share(&c) != 1 || c.callers != 0 ? "in the end" : nullptr;
}

int main(int argc, char** argv) {
  const std::string kind = argv[1];
  if (kind == "callers" || kind == "walk") {
    const char* e = kind == "walk" ? walk() : callers();
    return e ? failed(e, 0) : 0;
  }
  const unsigned long long seed0 = strtoull(argv[2], nullptr, 10);
  const int seeds = atoi(argv[3]);
  std::map<std::string, double> o{{"grid", 40}, {"hold", 0}, {"held", 0}, {"late", 0},
                                  {"levels", 60}, {"wide", 120}, {"small", 6}, {"wmax", 40},
                                  {"ticks", 0.02}, {"mode", 3}, {"path", 0}, {"k", 40}, {"stall", 0},
                                  {"join", 0}, {"after", 400000}, {"stripes", kSessStripes}};
  for (int i = 4; i < argc; ++i) {
    const std::string a = argv[i];
    const size_t eq = a.find('=');
    if (eq == a.npos || !o.count(a.substr(0, eq))) return failed("option", 0);
    o[a.substr(0, eq)] = atof(a.c_str() + eq + 1);
  }
  unsigned long long most = 0;
  for (unsigned long long seed = seed0; seed < seed0 + seeds; ++seed) {
    std::mt19937_64 rnd(seed);
    const Graph g = make(rnd, (int)o["levels"], (int)o["wide"], (int)o["wmax"],
                         (int)o["path"]);
    const int m = (int)g.col.size() - 1, s = 0;
    const bool weighted = kind == "weighted";
    const std::vector<int> want = search(g, s, weighted);
    long long reached = 0, edges = 0;
    for (int v = 0; v < g.n; ++v)
      if (want[v] >= 0) ++reached, edges += g.rp[v + 1] - g.rp[v];

    emu::Launch l;
    l.grid = (unsigned)o["grid"];
    l.block = kSB;
    l.seed = seed;
    l.hold = o["hold"];
    l.held_for = (unsigned)o["held"];
    l.ticks = o["ticks"];
    const double late = o["late"];
    std::vector<unsigned long long> start(l.grid, 0);
    for (unsigned b = 1; b < l.grid; ++b)
      if ((double)(rnd() % 1000) < late * 1000) start[b] = rnd() % (unsigned)o["after"];
    l.start = [&](unsigned b) { return start[b]; };

    if (kind == "batch") {
      const int k = (int)o["k"];
      l.stall_from = 15000;
      l.stall_to = l.stall_from + 1000000;
      const char* e = k > 64 ? batch<2>(g, k, l, o["stall"] > 0) : batch<1>(g, k, l, o["stall"] > 0);
      if (e) return failed(e, seed);
      continue;
    }
    std::vector<int> dist(g.n, -1);
    dist[s] = 0;
    const int nw = (g.n + 63) / 64;
    if (!weighted) {
      std::unique_ptr<SsspCtrl> ctrl(new SsspCtrl());
      std::unique_ptr<SessCtrl> sc(new SessCtrl());
      memset((void*)ctrl.get(), 0, sizeof(SsspCtrl));
      memset((void*)sc.get(), 0, sizeof(SessCtrl));
      std::vector<u64> vis0(nw, 0), vis1(nw, 0);
      vis0[0] = 1;
      std::vector<int> level_nf(g.n + 1);
      std::vector<uint8_t> dir(g.n + 1);
      SsspArgs a;
      memset(&a, 0, sizeof(a));
      a.n = g.n, a.nw = nw, a.m = m;
      a.rp = g.rp.data(), a.col = g.col.data(), a.ip = g.ip.data(), a.isrc = g.isrc.data();
      a.noin = g.noin.data(), a.vis0 = vis0.data(), a.vis1 = vis1.data();
      a.ctrl = ctrl.get(), a.dist = dist.data();
      a.mode = (int)o["mode"], a.alpha = 14, a.beta = 24, a.lane_edges = 4;
      a.small_edges = (int)o["small"];
      a.level_nf = level_nf.data(), a.level_dir = dir.data(), a.lrec = g.n + 1;
      Queues q(g, kHopPiece, sc.get(), s, (int)o["stripes"]);
      std::vector<std::unique_ptr<HopPolicy::Shared>> sh(l.grid);
      for (auto& p : sh) p.reset(new HopPolicy::Shared());
      const unsigned long long used =
          emu::run(l, [&](unsigned b) { session<HopPolicy>(a, q.x, *sh[b]); });
      if (!used) return failed("no end", seed);
      most = std::max(most, used);
      const LevelState& st = ctrl->st[1];
      if (st.done != 1) return failed("not done", seed);
      if (o["join"] > 0 && members<HopPolicy>(*sc) < l.grid) return failed("members", seed);
      if (st.reached != (u64)reached || st.source_edges != (u64)edges) return failed("totals", seed);
    } else {
      std::unique_ptr<WCtrl> ctrl(new WCtrl());
      memset((void*)ctrl.get(), 0, sizeof(WCtrl));
      std::vector<u64> fin(nw, 0), in0(nw, 0), in1(nw, 0);
      WArgs a;
      memset(&a, 0, sizeof(a));
      a.n = g.n, a.nw = nw, a.rp = g.rp.data();
      a.col = g.col.data(), a.wt = g.wt.data(), a.dist = dist.data();
      a.fin = fin.data(), a.inq[0] = in0.data(), a.inq[1] = in1.data(), a.ctrl = ctrl.get();
      int mx = 0;
      for (int w : g.wt) mx = std::max(mx, w);
      a.delta = 1 + (unsigned)(rnd() % 12);
      a.split = (int)a.delta < mx;
      std::vector<int> scol(g.col), swt(g.wt), light(g.n, 0);
      if (a.split && seed % 2) {                        // rows with the light edges first
        for (int v = 0; v < g.n; ++v) {
          std::vector<std::pair<int, int>> r;
          for (int i = g.rp[v]; i < g.rp[v + 1]; ++i) r.push_back({g.wt[i], g.col[i]});
          std::stable_partition(r.begin(), r.end(), [&](auto& x) { return x.first < (int)a.delta; });
          for (size_t i = 0; i < r.size(); ++i) {
            swt[g.rp[v] + i] = r[i].first, scol[g.rp[v] + i] = r[i].second;
            light[v] += r[i].first < (int)a.delta;
          }
        }
        a.col = scol.data(), a.wt = swt.data(), a.light = light.data();
      }
      a.half = (unsigned)(m / 2);
      a.max_rounds = (unsigned)(4 * g.n + 4);
      Queues q(g, kWeightPiece, &ctrl->sess, s, (int)o["stripes"]);
      std::vector<std::unique_ptr<WeightPolicy::Shared>> sh(l.grid);
      for (auto& p : sh) p.reset(new WeightPolicy::Shared()), p->low = 0;
      const unsigned long long used =
          emu::run(l, [&](unsigned b) { session<WeightPolicy>(a, q.x, *sh[b]); });
      if (!used) return failed("no end", seed);
      most = std::max(most, used);
      if (o["join"] > 0 && members<WeightPolicy>(ctrl->sess) < l.grid) return failed("members", seed);
      if (ctrl->done != 1) return failed(ctrl->done == 2 ? "too many levels" : "not done", seed);
    }
    if (dist != want) return failed("distances", seed);
  }
  printf("%d runs, at most %llu picks\n", seeds, most);
  return 0;
}
