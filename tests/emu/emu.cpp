#include "hip/hip_runtime.h"
#undef asm
#undef volatile

#include <stdio.h>
#include <sys/mman.h>

#include "emu.hpp"

// Saves the callee-saved registers on the running stack and goes on with another.
extern "C" void emu_switch(void** save, void* to);
__asm__(R"(
.text
.globl emu_switch
.type emu_switch,@function
emu_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
.size emu_switch,.-emu_switch
)");

namespace emu {

Idx tid, bid, gdim, bdim;

namespace {

constexpr size_t kStack = 48 << 10;
enum Where { kReady, kAtWave, kAtBlock, kPaused, kOver };

struct Lane {
  void* sp = nullptr;
  Where where = kReady;
  Op op = kMeet;
  unsigned long long x = 0, result = 0;
  int arg = 0, rows = 0;
};
struct Wave {
  unsigned block = 0, first = 0;    // first thread of it
  Lane lane[64];
  unsigned long long asleep = 0;    // not before this pick
};

std::vector<Wave> waves;
const std::function<void(unsigned)>* body;
Launch cfg;
void* scheduler;
Wave* wv;
Lane* ln;
unsigned long long picks;

void yield(Where w) {
  ln->where = w;
  emu_switch(&ln->sp, scheduler);
}
void enter() {
  (*body)(bid.x);
  yield(kOver);
  abort();
}

// One lane until it stops.
void go(Wave& w, unsigned l) {
  wv = &w;
  ln = &w.lane[l];
  tid = {w.first + l, 0, 0};
  bid = {w.block, 0, 0};
  gdim = {cfg.grid, 1, 1};
  bdim = {cfg.block, 1, 1};
  ln->where = kReady;
  emu_switch(&scheduler, ln->sp);
}

bool all(const Wave& w, Where x) {
  for (const Lane& l : w.lane)
    if (l.where != x && l.where != kOver) return false;
  return true;
}
bool over(const Wave& w) {
  for (const Lane& l : w.lane)
    if (l.where != kOver) return false;
  return true;
}

// The wave's lanes have all arrived: what each gets.
void meet(Wave& w) {
  unsigned long long votes = 0;
  const Op op = w.lane[0].op;
  for (int i = 0; i < 64; ++i) {
    if (w.lane[i].op != op) {
      fprintf(stderr, "lanes of a wave at different operations\n");
      abort();
    }
    if (w.lane[i].x & 1) votes |= 1ull << i;
  }
  for (int i = 0; i < 64; ++i) {
    Lane& l = w.lane[i];
    if (op == kBallot) l.result = votes;
    if (op == kShfl) l.result = w.lane[l.arg].x;
    if (op != kDpp) continue;
    int from = -1;
    if (l.arg > 0x110 && l.arg < 0x120) {               // row_shr
      const int n = l.arg - 0x110;
      if (i % 16 >= n) from = i - n;
    } else if (l.arg == 0x142) {                        // row_bcast:15
      if (i >= 16) from = i / 16 * 16 - 1;
    } else if (l.arg == 0x143) {                        // row_bcast:31
      if (i >= 32) from = 31;
    } else {
      abort();
    }
    if (!((l.rows >> (i / 16)) & 1)) from = -1;
    l.result = from < 0 ? 1ull << 32 : (unsigned long long)(unsigned)w.lane[from].x;
  }
  for (Lane& l : w.lane) l.where = kReady;
}

}  // namespace

unsigned long long wave_op(Op op, unsigned long long x, int arg, int rows) {
  ln->op = op;
  ln->x = x;
  ln->arg = arg;
  ln->rows = rows;
  Lane* me = ln;
  yield(kAtWave);
  return me->result;
}
void block_sync() { yield(kAtBlock); }
void pause() { yield(kPaused); }
unsigned long long clock() {
  double t = (double)picks;
  if (cfg.stalled >= 0 && picks > cfg.stall_from)
    t += (double)(picks - cfg.stall_from) * 1e5;
  return (unsigned long long)(t * cfg.ticks);
}

unsigned long long run(const Launch& l, const std::function<void(unsigned)>& kernel) {
  cfg = l;
  body = &kernel;
  picks = 0;
  const unsigned per = l.block / 64, n = l.grid * per;
  waves.assign(n, Wave());
  const size_t bytes = (size_t)n * 64 * kStack;
  char* mem = (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                          MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  for (unsigned i = 0; i < n; ++i) {
    waves[i].block = i / per;
    waves[i].first = i % per * 64;
    if (l.start) waves[i].asleep = l.start(i / per);
    for (int j = 0; j < 64; ++j) {
      void** sp = (void**)(mem + ((size_t)i * 64 + j + 1) * kStack);
      *--sp = nullptr;                       // keeps the stack as a call leaves it
      *--sp = (void*)&enter;
      for (int r = 0; r < 6; ++r) *--sp = nullptr;
      waves[i].lane[j].sp = sp;
    }
  }
  unsigned long long rng = l.seed * 0x9E3779B97F4A7C15ull + 1;
  auto draw = [&rng]() {
    rng ^= rng << 13;
    rng ^= rng >> 7;
    rng ^= rng << 17;
    return rng;
  };
  std::vector<unsigned> live(n);
  for (unsigned i = 0; i < n; ++i) live[i] = i;
  std::vector<unsigned> at_block(l.grid, 0), left(l.grid, per);
  while (!live.empty()) {
    if (++picks > l.limit) {
      munmap(mem, bytes);
      return 0;
    }
    const size_t at = draw() % live.size();
    const unsigned i = live[at];
    Wave& w = waves[i];
    if (picks < w.asleep || all(w, kAtBlock)) continue;
    if ((int)w.block == l.stalled && picks >= l.stall_from && picks < l.stall_to) continue;
    if (l.hold > 0 && (double)(draw() >> 11) / 9007199254740992.0 < l.hold)
      w.asleep = picks + l.held_for;
    for (int j = 63; j >= 0; --j)
      if (w.lane[j].where == kReady || w.lane[j].where == kPaused) go(w, (unsigned)j);
    if (over(w)) {
      live[at] = live.back();
      live.pop_back();
      --left[w.block];
    } else if (all(w, kAtWave)) {
      meet(w);
    } else if (all(w, kAtBlock)) {
      ++at_block[w.block];
    } else if (!all(w, kPaused)) {
      fprintf(stderr, "lanes of a wave at different places\n");
      abort();
    }
    const unsigned b = w.block;
    if (left[b] && at_block[b] == left[b]) {
      at_block[b] = 0;
      for (unsigned k = b * per; k < (b + 1) * per; ++k)
        for (Lane& x : waves[k].lane)
          if (x.where == kAtBlock) x.where = kReady;
    }
  }
  munmap(mem, bytes);
  return picks;
}

}  // namespace emu
