// Runs a block's threads one after the other on the CPU, in a chosen order
// between barriers, so that a kernel whose result depends on that order can be
// found without a GPU.  Stands in for <hip/hip_runtime.h> when the device part
// of a source file is compiled for the host: only what that part names is here.
#pragma once

#ifndef __HIP_PLATFORM_AMD__
#define __HIP_PLATFORM_AMD__
#endif
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <ucontext.h>

#include <algorithm>
#include <array>
#include <cstring>
#include <functional>
#include <memory>
#include <vector>

#undef __host__
#undef __device__
#undef __global__
#undef __shared__
#undef __forceinline__
#undef __launch_bounds__
#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...) unused

inline dim3 threadIdx, blockIdx, blockDim, gridDim;
using std::max;
using std::min;

namespace fiber {
constexpr int kWaveLanes = 64;
enum { kReady, kAtBlock, kAtWave, kGone };
struct Thread {
  ucontext_t ctx;
  std::vector<char> stack;
  int at = kReady;
};
inline std::vector<std::unique_ptr<Thread>> threads;
inline ucontext_t home;
inline int me = 0;
inline double exchange[1024 / kWaveLanes][kWaveLanes];
inline const std::function<void()>* body;

inline void stop(int at) {
  threads[me]->at = at;
  swapcontext(&threads[me]->ctx, &home);
}
inline void entry() {
  (*body)();
  stop(kGone);
}
// Runs f as block b of n threads; down: the highest thread first.
inline void run_block(int b, int n, bool down, const std::function<void()>& f) {
  body = &f;
  blockIdx = dim3(b, 0, 0);
  blockDim = dim3(n, 1, 1);
  threads.clear();
  for (int i = 0; i < n; ++i) {
    threads.emplace_back(new Thread());
    Thread& t = *threads.back();
    t.stack.resize(1 << 16);
    getcontext(&t.ctx);
    t.ctx.uc_stack.ss_sp = t.stack.data();
    t.ctx.uc_stack.ss_size = t.stack.size();
    t.ctx.uc_link = &home;
    makecontext(&t.ctx, entry, 0);
  }
  auto release = [&](int from, int to, int at) {   // all that still run have arrived
    int waiting = 0;
    for (int i = from; i < to; ++i) {
      if (threads[i]->at == kGone) continue;
      if (threads[i]->at != at) return;
      ++waiting;
    }
    if (waiting)
      for (int i = from; i < to; ++i)
        if (threads[i]->at == at) threads[i]->at = kReady;
  };
  for (bool live = true; live;) {
    live = false;
    for (int u = 0; u < n; ++u) {
      const int i = down ? n - 1 - u : u;
      if (threads[i]->at != kReady) continue;
      live = true;
      me = i;
      threadIdx = dim3(i, 0, 0);
      swapcontext(&home, &threads[i]->ctx);
    }
    for (int w = 0; w < n; w += kWaveLanes) release(w, std::min(n, w + kWaveLanes), kAtWave);
    release(0, n, kAtBlock);
    for (int i = 0; i < n; ++i) live = live || threads[i]->at == kReady;
  }
}
// The value that lane src(lane) of this wave passes.
template <class Src>
inline int from_lane(int v, Src src) {
  const int w = me / kWaveLanes, lane = me % kWaveLanes;
  exchange[w][lane] = v;
  stop(kAtWave);
  const int got = int(exchange[w][src(lane)]);
  stop(kAtWave);
  return got;
}
}  // namespace fiber

inline void __syncthreads() { fiber::stop(fiber::kAtBlock); }
inline int __double2loint(double d) { long long v; memcpy(&v, &d, 8); return int(v); }
inline int __double2hiint(double d) { long long v; memcpy(&v, &d, 8); return int(v >> 32); }
inline double __hiloint2double(int hi, int lo) {
  const long long v = (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo);
  double d;
  memcpy(&d, &v, 8);
  return d;
}
// both operands are the same value wherever the sources use these
inline std::array<int, 2> shim_swap(int v, int half) {
  const int lo = fiber::from_lane(v, [=](int l) { return l & ~half; });
  const int hi = fiber::from_lane(v, [=](int l) { return l | half; });
  return {lo, hi};
}
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) shim_swap(a, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) shim_swap(a, 16)
// row rotations (0x121 .. 0x12f) are the only controls that are run here
#define __builtin_amdgcn_update_dpp(old, v, ctrl, row, bank, bound) \
  fiber::from_lane(v, [](int l) { return (l & ~15) | ((l - ((ctrl) & 15)) & 15); })
template <typename V> inline V __shfl(V v, int, int = 64) { return v; }
template <typename V> inline V __shfl_up(V v, int, int = 64) { return v; }
template <typename V> inline V __shfl_down(V v, int, int = 64) { return v; }
template <typename V> inline V __shfl_xor(V v, int, int = 64) { return v; }
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_rcp(v) (1.0 / (v))
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_fetch_add(p, v, order, scope) (*(p) += (v), *(p) - (v))
#define __hip_atomic_load(p, order, scope) (*(p))
