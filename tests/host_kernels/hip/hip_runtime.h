// Just enough of the HIP device language, as plain C++, to run the format and pruning kernels on the
// CPU under the compiler's undefined-behaviour checks.  A workgroup's threads are fibers on one OS
// thread; a lane exchange is a switch to the next fiber, at which all fibers of a wave meet, a barrier as many as it takes until all
// fibers have come to it.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <ucontext.h>

#include <vector>

#define __global__ static
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ thread_local

struct uint2 { unsigned x, y; };
struct alignas(16) uint4 { unsigned x, y, z, w; };
struct alignas(16) int4 { int x, y, z, w; };
struct alignas(8) ushort4 { unsigned short x, y, z, w; };
inline uint2 make_uint2(unsigned x, unsigned y) { return {x, y}; }
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
inline ushort4 make_ushort4(unsigned short x, unsigned short y, unsigned short z, unsigned short w) { return {x, y, z, w}; }

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x = 1, unsigned y = 1, unsigned z = 1) : x(x), y(y), z(z) {}
};
inline dim3 blockIdx, threadIdx, blockDim, gridDim;

typedef int hipError_t;
typedef void* hipStream_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidConfiguration = 9;

namespace emu {
constexpr unsigned kMaxThreads = 256;
inline std::vector<char> stacks(kMaxThreads * (size_t)(256 << 10));
inline ucontext_t scheduler, fiber[kMaxThreads];
inline bool finished[kMaxThreads];
inline unsigned current;
inline unsigned barriers[kMaxThreads];              // that each fiber has come to
inline void* body;
inline void (*call)(void*);
inline unsigned long long slot[kMaxThreads];        // values of a lane exchange
inline hipError_t error = hipSuccess;
inline bool dry_run = false;                         // record launches, run nothing
inline unsigned long long launches, blocks;          // since the counters were last cleared

inline void fiber_main() {
  call(body);
  finished[current] = true;
  swapcontext(&fiber[current], &scheduler);
}
inline void yield() {
  const unsigned me = current;
  swapcontext(&fiber[me], &scheduler);
  threadIdx = dim3(me);
}
template <class F> void run_block(unsigned threads, F& f) {
  body = &f;
  call = [](void* p) { (*static_cast<F*>(p))(); };
  for (unsigned t = 0; t < threads; ++t) {
    getcontext(&fiber[t]);
    fiber[t].uc_stack.ss_sp = stacks.data() + t * (size_t)(256 << 10);
    fiber[t].uc_stack.ss_size = 256 << 10;
    fiber[t].uc_link = &scheduler;
    makecontext(&fiber[t], fiber_main, 0);
    finished[t] = false;
    barriers[t] = 0;
  }
  for (bool any = true; any;) {
    any = false;
    for (unsigned t = 0; t < threads; ++t)
      if (!finished[t]) {
        any = true;
        current = t;
        threadIdx = dim3(t);
        swapcontext(&scheduler, &fiber[t]);
      }
  }
}
// The runtime's own limits: 2^31-1 blocks and fewer than 2^32 threads along x, 65535 blocks along y.
template <class F> void launch(dim3 grid, dim3 block, F f) {
  if (grid.x == 0 || grid.y == 0 || grid.x >= (1u << 31) || (unsigned long long)grid.x * block.x >= (1ull << 32) || grid.y > 65535u) {
    error = hipErrorInvalidConfiguration;
    return;
  }
  ++launches;
  blocks += (unsigned long long)grid.x * grid.y;
  if (dry_run) return;
  gridDim = grid;
  blockDim = block;
  for (unsigned y = 0; y < grid.y; ++y)
    for (unsigned x = 0; x < grid.x; ++x) {
      blockIdx = dim3(x, y);
      run_block(block.x, f);
    }
}
}  // namespace emu

#define hipLaunchKernelGGL(fn, grid, block, lds, stream, ...) \
  emu::launch(grid, block, [=] { (void)(stream); (fn)(__VA_ARGS__); })
inline hipError_t hipGetLastError() {
  const hipError_t e = emu::error;
  emu::error = hipSuccess;
  return e;
}

inline void __syncthreads() {                          // (a wave may come to it many lane exchanges before another)
  const unsigned mine = ++emu::barriers[emu::current];
  for (bool wait = true; wait;) {
    emu::yield();
    wait = false;
    for (unsigned t = 0; t < blockDim.x; ++t) wait |= !emu::finished[t] && emu::barriers[t] < mine;
  }
}
template <class T> T __shfl_xor(T v, int mask) {
  emu::slot[emu::current] = v;
  emu::yield();
  const T other = (T)emu::slot[emu::current ^ (unsigned)mask];
  emu::yield();
  return other;
}
inline unsigned long long __ballot(bool x) {          // over the wave's threads that are still there
  emu::slot[emu::current] = x;
  emu::yield();
  unsigned long long lanes = 0;
  const unsigned wave = emu::current / 64 * 64;
  for (unsigned l = 0; l < 64 && wave + l < blockDim.x; ++l)
    if (!emu::finished[wave + l] && emu::slot[wave + l] != 0) lanes |= 1ull << l;
  emu::yield();
  return lanes;
}
template <class T> T atomicAdd(T* p, T v) { const T old = *p; *p = old + v; return old; }
template <class T> T atomicMin(T* p, T v) { const T old = *p; *p = old < v ? old : v; return old; }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
template <class T> T atomicMax(T* p, T v) { const T old = *p; *p = old > v ? old : v; return old; }
inline unsigned atomicOr(unsigned* p, unsigned v) { const unsigned old = *p; *p = old | v; return old; }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __ffs(int x) { return __builtin_ffs(x); }
inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
// bytes 0-3 are b's, 4-7 a's, 12 is zero
inline unsigned __builtin_amdgcn_perm(unsigned a, unsigned b, unsigned select) {
  const unsigned long long bytes = (unsigned long long)a << 32 | b;
  unsigned r = 0;
  for (int i = 0; i < 4; ++i) {
    const unsigned s = select >> (8 * i) & 0xff;
    if (s < 8) r |= (unsigned)(bytes >> (8 * s) & 0xff) << (8 * i);
    else if (s != 12) __builtin_trap();
  }
  return r;
}
// lane exchanges inside rows of 16 lanes: four lanes permuted, and the mirrored half row
inline unsigned __builtin_amdgcn_mov_dpp(unsigned v, int control, int, int, bool) {
  const unsigned l = emu::current;
  if (control < 0 || (control > 0xff && control != 0x141)) __builtin_trap();
  const unsigned from = control == 0x141 ? l / 8 * 8 + 7 - l % 8 : l / 4 * 4 + ((unsigned)control >> (2 * (l % 4)) & 3);
  emu::slot[l] = v;
  emu::yield();
  const unsigned other = (unsigned)emu::slot[from];
  emu::yield();
  return other;
}
