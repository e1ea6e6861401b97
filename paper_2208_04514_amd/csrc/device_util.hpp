// Wave64 and grid-level helpers for gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.hpp"

namespace dawn {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Mask of lanes below the calling lane.
__device__ __forceinline__ u64 lanes_below() {
  return (1ull << lane_id()) - 1ull;
}

__device__ __forceinline__ unsigned ld_acquire(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned ld_relaxed(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ld_relaxed(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Agent-scope relaxed stores: written through to the point every XCD reads
// coherently (a plain store may sit in its own XCD's L2 until the kernel ends).
__device__ __forceinline__ void st_relaxed(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ long long ld_relaxed(const long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned atom_add(unsigned* p, unsigned v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 atom_add(u64* p, u64 v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 atom_or(u64* p, u64 v) {
  return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One step of a wave-wide scan: the value the DPP control fetches from another
// lane, 0 where it fetches none.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_get(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum across the wave (every lane takes part): four shifts
// within rows of 16 lanes, then the rows' totals broadcast to later rows.  Six
// VALU instructions with no LDS in the chain; the same scan by six dependent
// lane permutes takes about 0.2 us, and a level has several on its way.
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += dpp_get<0x111, 0xf>(x);   // row_shr:1
  x += dpp_get<0x112, 0xf>(x);   // row_shr:2
  x += dpp_get<0x114, 0xf>(x);   // row_shr:4
  x += dpp_get<0x118, 0xf>(x);   // row_shr:8
  x += dpp_get<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  x += dpp_get<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Inclusive prefix maximum across the wave of values >= 0.
__device__ __forceinline__ int wave_incl_max(int x) {
  x = max(x, dpp_get<0x111, 0xf>(x));
  x = max(x, dpp_get<0x112, 0xf>(x));
  x = max(x, dpp_get<0x114, 0xf>(x));
  x = max(x, dpp_get<0x118, 0xf>(x));
  x = max(x, dpp_get<0x142, 0xa>(x));
  x = max(x, dpp_get<0x143, 0xc>(x));
  return x;
}

// Sums across the wave (every lane takes part), the same in every lane.
__device__ __forceinline__ unsigned wave_sum(unsigned x) {
  return (unsigned)__builtin_amdgcn_readlane(wave_incl_scan((int)x), kWave - 1);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ u64 dpp_get64(u64 x) {
  const unsigned lo = (unsigned)dpp_get<CTRL, ROWS>((int)(unsigned)x);
  const unsigned hi = (unsigned)dpp_get<CTRL, ROWS>((int)(unsigned)(x >> 32));
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 wave_sum(u64 x) {
  x += dpp_get64<0x111, 0xf>(x);
  x += dpp_get64<0x112, 0xf>(x);
  x += dpp_get64<0x114, 0xf>(x);
  x += dpp_get64<0x118, 0xf>(x);
  x += dpp_get64<0x142, 0xa>(x);
  x += dpp_get64<0x143, 0xc>(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, kWave - 1);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), kWave - 1);
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 wave_or(u64 x) {
  x |= dpp_get64<0x111, 0xf>(x);
  x |= dpp_get64<0x112, 0xf>(x);
  x |= dpp_get64<0x114, 0xf>(x);
  x |= dpp_get64<0x118, 0xf>(x);
  x |= dpp_get64<0x142, 0xa>(x);
  x |= dpp_get64<0x143, 0xc>(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, kWave - 1);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), kWave - 1);
  return ((u64)hi << 32) | lo;
}

// Smallest j in [0, 64) with incl[j] > x, where `incl` is the wave's
// non-decreasing inclusive scan and incl[63] > x.  Six lane permutes.
__device__ __forceinline__ int wave_owner(int incl, int x) {
  int lo = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1) {
    int probe = lo + step - 1;
    int v = __shfl(incl, probe, kWave);
    if (v <= x) lo = probe + 1;
  }
  return lo;
}

// Wave-aggregated append: every lane with `pred` gets a distinct slot from
// *counter; one atomic per wave.  Returns the slot, or -1 without `pred`.
__device__ __forceinline__ int wave_append(unsigned* counter, bool pred) {
  u64 mask = __ballot(pred);
  if (mask == 0) return -1;
  int leader = __ffsll((unsigned long long)mask) - 1;
  unsigned base = 0;
  if (lane_id() == leader) base = atom_add(counter, (unsigned)__popcll(mask));
  base = __shfl(base, leader, kWave);
  return pred ? (int)(base + __popcll(mask & lanes_below())) : -1;
}

// Block-wide sums, one call per counter set; every thread must call it.
template <int BLOCK>
__device__ __forceinline__ void block_sum3(unsigned& a, u64& b, u64& c) {
  __shared__ unsigned sa[BLOCK / kWave];
  __shared__ u64 sb[BLOCK / kWave], sc[BLOCK / kWave];
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int w = threadIdx.x / kWave;
  __syncthreads();
  if (lane_id() == 0) { sa[w] = a; sb[w] = b; sc[w] = c; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < BLOCK / kWave; ++i) { a += sa[i]; b += sb[i]; c += sc[i]; }
  }
  __syncthreads();
}

// Barrier across all workgroups of a cooperative launch.  Thread 0 of each
// workgroup arrives with a release fence and waits with an acquire fence at
// agent scope, so plain stores before the barrier are visible to plain loads
// after it on every XCD.  The last arriver resets the count and bumps the
// generation, so the state is reusable across barriers and launches.
//
// The wait is bounded: after kBarrierTimeoutTicks of the 100 MHz wall clock a
// waiter raises `abort` and leaves, and every later call returns false at
// once, so a kernel always drains even if its workgroups ever disagreed on the
// number of barriers.  Returns false on abort.
constexpr unsigned long long kBarrierTimeoutTicks = 1000000000ull;   // 10 s

__device__ __forceinline__ bool grid_sync(GridBarrier* bar) {
  __shared__ int ok;
  __syncthreads();
  if (gridDim.x == 1) return true;   // one workgroup: the workgroup barrier is enough
  if (threadIdx.x == 0) {
    ok = 1;
    const unsigned nb = gridDim.x;
    if (__hip_atomic_load(&bar->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      ok = 0;
    } else {
      unsigned g = __hip_atomic_load(&bar->gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __threadfence();
      unsigned arrived = __hip_atomic_fetch_add(&bar->count, 1u, __ATOMIC_ACQ_REL,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (arrived == nb - 1) {
        __hip_atomic_store(&bar->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&bar->gen, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        const unsigned long long t0 = wall_clock64();
        while (__hip_atomic_load(&bar->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
          if (__hip_atomic_load(&bar->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
              wall_clock64() - t0 > kBarrierTimeoutTicks) {
            __hip_atomic_store(&bar->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = 0;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      __threadfence();
    }
  }
  __syncthreads();
  return ok != 0;
}

}  // namespace dawn
