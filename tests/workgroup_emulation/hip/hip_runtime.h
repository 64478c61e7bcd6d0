// One GPU workgroup on the CPU, for tests of the kernels' barriers: the kernel sources
// are compiled as host code against this header, every thread of a workgroup is a
// coroutine, and waves run as far ahead of each other as the barriers let them, in an
// order the test chooses. Only what the lattice passes use is here.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <cmath>
#include <functional>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(n)
#define __align__(n) __attribute__((aligned(n)))
#define amdgpu_waves_per_eu(...) unused

struct dim3 {
  unsigned x, y, z;
};
struct float4 {
  float x, y, z, w;
};
struct double2 {
  double x, y;
};
struct uint4 {
  unsigned x, y, z, w;
};
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return uint4{x, y, z, w}; }

template <class T>
inline T min(T a, T b) { return b < a ? b : a; }
template <class T>
inline T max(T a, T b) { return a < b ? b : a; }
inline float fabs(float x) { return ::fabsf(x); }
inline float fmax(float a, float b) { return ::fmaxf(a, b); }
inline float sqrt(float x) { return ::sqrtf(x); }
inline float fma(float a, float b, float c) { return ::fmaf(a, b, c); }
using std::isfinite;

inline long long __double_as_longlong(double x) {
  long long r;
  memcpy(&r, &x, 8);
  return r;
}
inline double __longlong_as_double(long long x) {
  double r;
  memcpy(&r, &x, 8);
  return r;
}

namespace emu {

constexpr int kWave = 64, kMaxThreads = 1024, kStack = 128 * 1024;

struct Thread {
  ucontext_t ctx;
  std::vector<char> stack;
  dim3 tid;
  bool done = true;
  unsigned posts = 0;  // lane exchanges of the thread so far
};

struct Group {
  Thread t[kMaxThreads];
  int n = 0, cur = 0, live = 0;
  long progress = 0;
  int at_barrier = 0;
  unsigned barriers = 0;  // barriers passed by the workgroup
  unsigned lane[kMaxThreads / kWave][2][kWave], posted[kMaxThreads / kWave] = {};
  ucontext_t sched;
  std::function<void()> kernel;
};
inline Group g;

inline void yield() { swapcontext(&g.t[g.cur].ctx, &g.sched); }

// A barrier opens between two turns of the waves (run()), so that the lanes of a wave
// pass it together.
inline void barrier() {
  const unsigned gen = g.barriers;
  ++g.at_barrier;
  ++g.progress;
  while (g.barriers == gen) yield();
}

// x of every lane of the wave, once all 64 have given theirs
inline const unsigned* exchange(unsigned x) {
  Thread& t = g.t[g.cur];
  const int w = g.cur / kWave;
  unsigned* slot = g.lane[w][t.posts & 1];
  slot[g.cur % kWave] = x;
  ++t.posts;
  ++g.posted[w];
  ++g.progress;
  while (g.posted[w] < kWave * t.posts) yield();
  return slot;
}

inline int lane() { return g.cur % kWave; }

struct Swap {
  unsigned r[2];
  unsigned operator[](int k) const { return r[k]; }
};
// lane swaps of a value with itself: both halves of the pair (i, i ^ o)
inline Swap swap_self(unsigned x, int o) {
  const unsigned* v = exchange(x);
  return Swap{{v[lane() & ~o], v[lane() | o]}};
}
inline int dpp(int x, int ctrl) {
  const unsigned* v = exchange((unsigned)x);
  const int l = lane();
  if (ctrl >= 0x121 && ctrl <= 0x12F) return (int)v[(l & ~15) | ((l - (ctrl - 0x120)) & 15)];  // rotate a row right
  return (int)v[(l & ~3) | ((ctrl >> (2 * (l & 3))) & 3)];                                     // permute a quad
}

inline void entry() {
  g.kernel();
  Thread& t = g.t[g.cur];
  t.done = true;
  --g.live;
  ++g.progress;
  while (true) yield();
}

// Workgroup b of a grid: the kernel called by every thread. order: the waves, the one
// that runs furthest ahead first. False if the workgroup hangs.
inline bool run(dim3 blockDim_, dim3 gridDim_, unsigned b, const std::vector<int>& order, std::function<void()> kernel);

}  // namespace emu

#define threadIdx (emu::g.t[emu::g.cur].tid)
inline dim3 blockIdx, blockDim, gridDim;
inline void __syncthreads() { emu::barrier(); }

#define __builtin_amdgcn_readfirstlane(x) ((int)emu::exchange((unsigned)(x))[0])
#define __builtin_amdgcn_permlane32_swap(x, y, fi, bc) emu::swap_self(x, 32)
#define __builtin_amdgcn_permlane16_swap(x, y, fi, bc) emu::swap_self(x, 16)
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rm, bm, bc) emu::dpp(x, ctrl)

inline bool emu::run(dim3 bd, dim3 gd, unsigned b, const std::vector<int>& order, std::function<void()> kernel) {
  blockDim = bd;
  gridDim = gd;
  blockIdx = dim3{b, 0, 0};
  g.n = g.live = (int)(bd.x * bd.y);
  g.kernel = kernel;
  g.at_barrier = 0;
  memset(g.posted, 0, sizeof(g.posted));
  for (int i = 0; i < g.n; ++i) {
    Thread& t = g.t[i];
    t.stack.resize(kStack);
    t.tid = dim3{i % bd.x, i / bd.x, 0};
    t.done = false;
    t.posts = 0;
    getcontext(&t.ctx);
    t.ctx.uc_stack.ss_sp = t.stack.data();
    t.ctx.uc_stack.ss_size = kStack;
    t.ctx.uc_link = nullptr;
    makecontext(&t.ctx, entry, 0);
  }
  while (g.live) {
    bool moved = false;
    if (g.at_barrier == g.live) {
      g.at_barrier = 0;
      ++g.barriers;
    }
    for (size_t k = 0; k < order.size() && !moved; ++k) {  // after a move the first wave is tried again
      const long p = g.progress;
      for (int i = order[k] * kWave; i < (order[k] + 1) * kWave; ++i) {
        if (g.t[i].done) continue;
        g.cur = i;
        swapcontext(&g.sched, &g.t[i].ctx);
      }
      moved = g.progress != p;
    }
    if (!moved) return false;
  }
  return true;
}
