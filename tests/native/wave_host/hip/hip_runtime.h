// A host execution model of wave64 kernels, for tests only. In front of the
// ROCm headers on the include path it lets clang compile the library's sources
// as plain C++, so that a kernel's logic can be checked without a GPU, and in
// orders that the hardware is free to choose but hardly ever does.
//
// A workgroup's threads are fibers. A wave runs until all of its lanes wait at
// a barrier or have ended; a lane runs until the next operation that its wave
// takes together (shuffle, ballot, wave barrier), where lanes meet. Waves take
// turns in ascending or descending order, and so do workgroups: two writes to
// one place with no barrier between them land in either order.
// Not modelled: caches, memory ordering, timing, divergent wave operations of
// different kinds (an error).
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __shared__ static
#define __align__(x) __attribute__((aligned(x)))
#define __launch_bounds__(...)

struct dim3 {
  uint32_t x, y, z;
  constexpr dim3(uint32_t a = 1, uint32_t b = 1, uint32_t c = 1)
      : x(a), y(b), z(c) {}
};
struct __attribute__((aligned(8))) uint2 { uint32_t x, y; };
struct __attribute__((aligned(16))) uint4 { uint32_t x, y, z, w; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return uint2{x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
  return uint4{x, y, z, w};
}

inline dim3 threadIdx, blockIdx, gridDim, blockDim;

namespace wave_host {

enum State { kReady, kAtWave, kAtBlock, kDone };
constexpr uint32_t kMaxThreads = 1024;
constexpr size_t kStack = 128 * 1024;

struct Fiber {
  ucontext_t ctx;
  State state;
  int kind;      // the wave operation it waits at
  uint64_t val;  // what it brings there
};
struct Exchange {
  uint64_t val[64];
  uint64_t active;
};

inline Fiber fibers[kMaxThreads];
inline Exchange exchange[kMaxThreads / 64];
inline ucontext_t scheduler;
inline uint32_t current;
inline void (*body)(void *);
inline void *body_arg;
inline char *stacks;
inline bool waves_descend, groups_descend;
inline uint32_t max_groups = ~0u;  // run only this many of a launch's groups
inline uint32_t launches, groups_launched;  // since they were last cleared
inline void *last_kernel;

inline void yield(State s) {
  Fiber &f = fibers[current];
  f.state = s;
  swapcontext(&f.ctx, &scheduler);
}

inline void entry() {
  body(body_arg);
  fibers[current].state = kDone;
  swapcontext(&fibers[current].ctx, &scheduler);
}

inline void resume(uint32_t t) {
  current = t;
  threadIdx = dim3(t);
  swapcontext(&scheduler, &fibers[t].ctx);
}

// Every lane of the wave brings v; returns what the active lanes brought.
inline const Exchange &meet(int kind, uint64_t v) {
  Fiber &f = fibers[current];
  f.kind = kind;
  f.val = v;
  yield(kAtWave);
  return exchange[current >> 6];
}

// Runs wave w until its lanes are at a barrier or done.
inline void run_wave(uint32_t w, uint32_t threads) {
  const uint32_t lo = w * 64, hi = lo + 64 < threads ? lo + 64 : threads;
  for (;;) {
    for (uint32_t t = lo; t < hi; ++t)
      if (fibers[t].state == kReady) resume(t);
    Exchange x{};
    int kind = -1;
    for (uint32_t t = lo; t < hi; ++t) {
      Fiber &f = fibers[t];
      if (f.state != kAtWave) continue;
      if (kind >= 0 && f.kind != kind) {
        fprintf(stderr, "wave_host: lanes at different wave operations\n");
        abort();
      }
      kind = f.kind;
      x.val[t - lo] = f.val;
      x.active |= 1ull << (t - lo);
      f.state = kReady;
    }
    if (kind < 0) return;
    exchange[w] = x;
  }
}

inline void run_group(uint32_t threads) {
  if (threads > kMaxThreads) abort();
  if (!stacks) {
    stacks = static_cast<char *>(mmap(nullptr, kStack * kMaxThreads,
                                      PROT_READ | PROT_WRITE,
                                      MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    if (stacks == MAP_FAILED) abort();
  }
  for (uint32_t t = 0; t < threads; ++t) {
    Fiber &f = fibers[t];
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = stacks + size_t(t) * kStack;
    f.ctx.uc_stack.ss_size = kStack;
    f.ctx.uc_link = nullptr;
    makecontext(&f.ctx, entry, 0);
    f.state = kReady;
  }
  const uint32_t waves = (threads + 63) / 64;
  for (bool any = true; any;) {
    for (uint32_t i = 0; i < waves; ++i)
      run_wave(waves_descend ? waves - 1 - i : i, threads);
    any = false;
    for (uint32_t t = 0; t < threads; ++t)
      if (fibers[t].state == kAtBlock) {
        fibers[t].state = kReady;
        any = true;
      }
  }
}

inline uint32_t lane_id() { return threadIdx.x & 63u; }

template <typename T>
inline T from_lane(int kind, T v, uint32_t src) {
  uint64_t u = 0;
  memcpy(&u, &v, sizeof v);
  u = meet(kind, u).val[src & 63u];
  memcpy(&v, &u, sizeof v);
  return v;
}

}  // namespace wave_host

// ---- workgroup and wave operations ----
inline void __syncthreads() { wave_host::yield(wave_host::kAtBlock); }
inline void __builtin_wave_host_barrier() { wave_host::meet(0, 0); }
#define __builtin_amdgcn_wave_barrier __builtin_wave_host_barrier
#define __builtin_amdgcn_fence(...) ((void)0)

inline uint64_t __ballot(int p) {
  const wave_host::Exchange &x = wave_host::meet(1, p != 0);
  uint64_t m = 0;
  for (int i = 0; i < 64; ++i) m |= (x.val[i] & 1ull) << i;
  return m & x.active;
}
template <typename T>
inline T __shfl(T v, int src, int) {
  return wave_host::from_lane(2, v, uint32_t(src));
}
template <typename T>
inline T __shfl_xor(T v, int mask, int) {
  return wave_host::from_lane(3, v, wave_host::lane_id() ^ uint32_t(mask));
}
template <typename T>
inline T __shfl_up(T v, uint32_t d, int) {
  const uint32_t l = wave_host::lane_id();
  const T o = wave_host::from_lane(4, v, l >= d ? l - d : l);
  return l >= d ? o : v;
}
inline int wave_host_readlane(int v, int lane) {
  return wave_host::from_lane(5, v, uint32_t(lane));
}
inline uint32_t wave_host_readfirstlane(uint32_t v) {
  const wave_host::Exchange &x = wave_host::meet(6, v);
  return uint32_t(x.val[__builtin_ctzll(x.active)]);
}
// row_shr:1 ... 15 (0x111 ... 0x11F), row_bcast:15 (0x142), row_bcast:31
// (0x143); row masks by rows of 16 lanes, every bank
inline int wave_host_dpp(int old, int v, int ctrl, int row_mask, int,
                         bool bound_ctrl) {
  const wave_host::Exchange &x = wave_host::meet(7, uint32_t(v));
  const uint32_t l = wave_host::lane_id(), row = l >> 4;
  if (!((row_mask >> row) & 1)) return old;
  if (ctrl == 0x142) return row ? int(x.val[row * 16 - 1]) : old;
  if (ctrl == 0x143) return l >= 32 ? int(x.val[31]) : old;
  const uint32_t s = uint32_t(ctrl) & 15u;
  if ((ctrl & ~15) != 0x110 || s == 0) abort();
  if ((l & 15u) < s) return bound_ctrl ? 0 : old;
  return int(x.val[l - s]);
}
#define __builtin_amdgcn_readlane wave_host_readlane
#define __builtin_amdgcn_readfirstlane wave_host_readfirstlane
#define __builtin_amdgcn_update_dpp wave_host_dpp

// ---- lane operations ----
inline uint32_t wave_host_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  const uint64_t both = (uint64_t(hi) << 32) | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = (sel >> (8 * i)) & 255u;
    if (s > 7) abort();
    r |= (uint32_t(both >> (8 * s)) & 255u) << (8 * i);
  }
  return r;
}
inline uint32_t wave_host_mbcnt_lo(uint32_t m, uint32_t base) {
  const uint32_t l = wave_host::lane_id();
  return base + uint32_t(__builtin_popcount(
                    l < 32 ? m & ((1u << l) - 1u) : m));
}
inline uint32_t wave_host_mbcnt_hi(uint32_t m, uint32_t base) {
  const uint32_t l = wave_host::lane_id();
  return base + (l < 32 ? 0u
                        : uint32_t(__builtin_popcount(
                              m & ((1u << (l - 32)) - 1u))));
}
#define __builtin_amdgcn_perm wave_host_perm
#define __builtin_amdgcn_mbcnt_lo wave_host_mbcnt_lo
#define __builtin_amdgcn_mbcnt_hi wave_host_mbcnt_hi
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __clz(int v) { return v ? __builtin_clz(uint32_t(v)) : 32; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) {
  return uint32_t((uint64_t(a) * b) >> 32);
}
inline uint32_t __umul24(uint32_t a, uint32_t b) {
  return (a & 0xFFFFFFu) * (b & 0xFFFFFFu);
}
template <typename T>
inline T min(T a, T b) { return b < a ? b : a; }
template <typename T>
inline T max(T a, T b) { return a < b ? b : a; }
inline uint32_t atomicAdd(uint32_t *p, uint32_t v) {
  const uint32_t o = *p;
  *p = o + v;
  return o;
}
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_fetch_or(p, v, order, scope) (*(p) |= (v))

// ---- the runtime calls of the library ----
typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidDevice = 101 };
enum { hipMemcpyDeviceToHost = 2 };
#define HIP_SYMBOL(x) (x)
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int,
                                 hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
inline hipError_t hipGetSymbolAddress(void **p, void *sym) {
  return *p = sym, hipSuccess;
}

template <typename... P, typename... A>
void hipLaunchKernelGGL(void (*k)(P...), dim3 grid, dim3 block, uint32_t,
                        hipStream_t, A... args) {
  auto call = [&] { k(static_cast<P>(args)...); };
  using Call = decltype(call);
  wave_host::body = [](void *p) { (*static_cast<Call *>(p))(); };
  wave_host::body_arg = &call;
  gridDim = grid;
  blockDim = block;
  const uint64_t groups = uint64_t(grid.x) * grid.y;
  ++wave_host::launches;
  wave_host::last_kernel = reinterpret_cast<void *>(k);
  wave_host::groups_launched += uint32_t(groups);
  for (uint64_t i = 0; i < groups && i < wave_host::max_groups; ++i) {
    const uint64_t g = wave_host::groups_descend ? groups - 1 - i : i;
    blockIdx = dim3(uint32_t(g % grid.x), uint32_t(g / grid.x));
    wave_host::run_group(block.x);
  }
}
