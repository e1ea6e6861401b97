// A stand-in for the HIP runtime's header that runs device code on the host: one
// fiber per lane, 64 lanes to a wave, wave operations as meeting points of its
// lanes (emu.cpp).  Between two meeting points a wave's lanes run one after
// another, lane 0 last: what lane 0 writes comes after what the others read before
// it, as in lockstep; the other order has to be made by a wave barrier.
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

using std::max;
using std::min;

// ------------------------------------------------------------------ host side --
typedef int hipError_t;
constexpr int hipSuccess = 0, hipErrorNotReady = 600;
typedef struct emu_stream* hipStream_t;
typedef struct emu_event* hipEvent_t;
typedef struct emu_graph* hipGraphExec_t;
constexpr unsigned hipHostMallocCoherent = 1, hipHostMallocMapped = 2, hipStreamNonBlocking = 1,
                   hipEventDisableTiming = 2;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
inline const char* hipGetErrorString(hipError_t) { return "emulated"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
template <class F>
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, F, int, size_t) {
  *n = 1;
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipSuccess; }
inline hipError_t hipHostFree(void*) { return hipSuccess; }
inline hipError_t hipHostMalloc(void**, size_t, unsigned) { return hipSuccess; }
inline hipError_t hipHostGetDevicePointer(void**, void*, unsigned) { return hipSuccess; }
#define hipLaunchKernelGGL(...) ((void)0)

// ---------------------------------------------------------------- device side --
#define __device__
#define __global__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)

namespace emu {
struct Idx {
  unsigned x, y, z;
};
extern Idx tid, bid, gdim, bdim;      // of the lane that runs
enum Op { kBallot, kShfl, kDpp, kMeet };
// All lanes of the wave come here; lane l gets what `op` gives it.
unsigned long long wave_op(Op op, unsigned long long x, int arg, int rows);
void block_sync();
void pause();
unsigned long long clock();
}  // namespace emu

#define threadIdx emu::tid
#define blockIdx emu::bid
#define gridDim emu::gdim
#define blockDim emu::bdim
inline unsigned __lane_id() { return emu::tid.x & 63u; }
inline void __syncthreads() { emu::block_sync(); }
inline unsigned long long __ballot(bool p) { return emu::wave_op(emu::kBallot, p, 0, 0); }
template <class T>
T __shfl(T x, int lane, int = 64) {
  return (T)emu::wave_op(emu::kShfl, (unsigned long long)(unsigned)x, lane & 63, 0);
}
template <class T>
T __shfl_xor(T x, int m, int = 64) {
  return __shfl(x, (int)__lane_id() ^ m);
}
inline int emu_dpp(int old, int x, int ctrl, int rows) {
  const unsigned long long r = emu::wave_op(emu::kDpp, (unsigned)x, ctrl, rows);
  return r >> 32 ? old : (int)(unsigned)r;
}
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, bound) emu_dpp(old, x, ctrl, rows)
inline int __builtin_amdgcn_readlane(int x, int lane) { return __shfl(x, lane); }
inline int __builtin_amdgcn_readfirstlane(int x) { return __shfl(x, 0); }
inline void __builtin_amdgcn_wave_barrier() { emu::wave_op(emu::kMeet, 0, 0, 0); }
#define __builtin_amdgcn_fence(order, scope) ((void)0)
inline void __builtin_amdgcn_s_sleep(int) { emu::pause(); }
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline void __threadfence() {}
inline unsigned long long wall_clock64() { return emu::clock(); }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline int __ffsll(unsigned long long x) { return __builtin_ffsll((long long)x); }
inline int __clz(int x) { return x ? __builtin_clz((unsigned)x) : 32; }

#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 1
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_store(p, v, o, s) ((void)(*(p) = (v)))
template <class T, class V, class F>
T emu_rmw(T* p, V v, F f) {
  const T old = *p;
  *p = f(old, (T)v);
  return old;
}
#define __hip_atomic_fetch_add(p, v, o, s) emu_rmw(p, v, [](auto a, auto b) { return a + b; })
#define __hip_atomic_fetch_or(p, v, o, s) emu_rmw(p, v, [](auto a, auto b) { return a | b; })
#define __hip_atomic_fetch_and(p, v, o, s) emu_rmw(p, v, [](auto a, auto b) { return a & b; })
#define __hip_atomic_fetch_min(p, v, o, s) emu_rmw(p, v, [](auto a, auto b) { return min(a, b); })
#define __hip_atomic_fetch_max(p, v, o, s) emu_rmw(p, v, [](auto a, auto b) { return max(a, b); })
template <class T, class V>
T atomicAdd(T* p, V v) { return __hip_atomic_fetch_add(p, v, 0, 0); }
template <class T, class V>
T atomicOr(T* p, V v) { return __hip_atomic_fetch_or(p, v, 0, 0); }
template <class T, class V>
T atomicAnd(T* p, V v) { return __hip_atomic_fetch_and(p, v, 0, 0); }
template <class T, class V>
T atomicMax(T* p, V v) { return __hip_atomic_fetch_max(p, v, 0, 0); }

// asm volatile("s_waitcnt ...") and the like: nothing to wait for
#define asm
#define volatile(...)
