// One workgroup at a time on the host, its threads as fibers of one OS thread: enough of the
// device language to run the solver's vector kernels unchanged.  The caller decides when the
// waves of a workgroup start (Gate), and so in which order they read memory.
#pragma once

#include <hip/hip_runtime_api.h>
#include <ucontext.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <vector>

#undef __global__
#undef __device__
#undef __host__
#undef __shared__
#undef __forceinline__
#undef __launch_bounds__
#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 0

namespace emulate {

struct Index {
  unsigned x = 0, y = 0, z = 0;
};
inline Index thread, block, block_size, grid_size;

// Workgroup `block`: the waves for which held(wave) is true start only when all others wait at
// a barrier (or have ended), after `between` has run.
struct Gate {
  int block = -1;
  std::function<bool(int)> held;
  std::function<void()> between;
};
inline Gate gate;

enum State { kReady, kWave, kBarrier, kHeld, kEnded };
struct Fiber {
  ucontext_t ctx;
  std::vector<char> stack;
  State state;
  int shuffles;  // shuffles so far: their buffers alternate
};
inline std::vector<Fiber> fibers;
inline ucontext_t scheduler;
inline int current;
inline double shuffle_buf[2][1024];
inline std::function<void()> body;

inline void wait_for(State s) {
  fibers[size_t(current)].state = s;
  const int me = current;
  swapcontext(&fibers[size_t(me)].ctx, &scheduler);
}
inline void entry() {
  body();
  fibers[size_t(current)].state = kEnded;
  swapcontext(&fibers[size_t(current)].ctx, &scheduler);
}

inline void run_block(int n, const Gate* g) {
  fibers.resize(size_t(n));
  for (int t = 0; t < n; ++t) {
    Fiber& f = fibers[size_t(t)];
    f.stack.resize(64 * 1024);
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = f.stack.data();
    f.ctx.uc_stack.ss_size = f.stack.size();
    f.ctx.uc_link = &scheduler;
    makecontext(&f.ctx, entry, 0);
    f.shuffles = 0;
    f.state = g && g->held(t / 64) ? kHeld : kReady;
  }
  auto all = [&](int a, int b, State s) {  // every thread of [a, b) that has not ended is in s
    bool any = false;
    for (int t = a; t < b; ++t) {
      if (fibers[size_t(t)].state == kEnded) continue;
      if (fibers[size_t(t)].state != s) return false;
      any = true;
    }
    return any;
  };
  auto ready = [&](int a, int b) {
    for (int t = a; t < b; ++t)
      if (fibers[size_t(t)].state != kEnded) fibers[size_t(t)].state = kReady;
  };
  while (true) {
    bool ran = false;
    for (int t = 0; t < n; ++t)
      if (fibers[size_t(t)].state == kReady) {
        ran = true;
        current = t;
        thread.x = unsigned(t);
        swapcontext(&scheduler, &fibers[size_t(t)].ctx);
      }
    for (int w = 0; w < n; w += 64)
      if (all(w, std::min(n, w + 64), kWave)) {
        ready(w, std::min(n, w + 64));
        ran = true;
      }
    if (ran) continue;
    bool held = false;
    for (Fiber& f : fibers) held = held || f.state == kHeld;
    if (held) {
      g->between();
      for (Fiber& f : fibers)
        if (f.state == kHeld) f.state = kReady;
    } else if (all(0, n, kBarrier)) {
      ready(0, n);
    } else {
      return;  // all have ended
    }
  }
}

template <typename F>
void launch(dim3 grid, dim3 threads, F f) {
  grid_size = {grid.x, grid.y, grid.z};
  block_size = {threads.x, threads.y, threads.z};
  body = f;
  for (unsigned b = 0; b < grid.x; ++b) {
    block.x = b;
    run_block(int(threads.x), int(b) == gate.block ? &gate : nullptr);
  }
}

}  // namespace emulate

#define threadIdx emulate::thread
#define blockIdx emulate::block
#define blockDim emulate::block_size
#define gridDim emulate::grid_size
#define hipLaunchKernelGGL(kernel, grid, threads, lds, stream, ...) \
  emulate::launch(grid, threads, [&] { kernel(__VA_ARGS__); })
#define hipGetLastError() hipSuccess
#define hipGetErrorString(e) "error"

inline void __syncthreads() { emulate::wait_for(emulate::kBarrier); }
inline void __threadfence() {}
inline double __shfl_xor(double v, int off, int) {
  emulate::Fiber& f = emulate::fibers[size_t(emulate::current)];
  double* const buf = emulate::shuffle_buf[f.shuffles++ & 1];
  buf[emulate::current] = v;
  emulate::wait_for(emulate::kWave);
  return buf[emulate::current ^ off];
}
template <typename T>
T emulate_load(const T* p) {
  return *p;
}
#define __hip_atomic_load(p, order, scope) emulate_load(p)
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
inline uint32_t atomicAdd(uint32_t* p, uint32_t v) {
  const uint32_t old = *p;
  *p += v;
  return old;
}
inline uint32_t __builtin_amdgcn_readfirstlane(uint32_t v) { return v; }
inline uint32_t __float_as_uint(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  return u;
}
using std::isfinite;
using std::min;
