// Stands in for the HIP header when a kernel source is compiled for the CPU:
// one block at a time, every thread a fiber. The lanes of a wave meet at each
// cross-lane operation and the block at each barrier, so code whose cross-lane
// operations are reached by whole waves runs as on the GPU, in an order that
// is the same every time.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <memory>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define hipLaunchKernelGGL(...) ((void)0)

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0 };
inline hipError_t hipGetLastError() { return hipSuccess; }

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };

using std::max;
using std::min;

namespace hip_host {

constexpr int kLanes = 64;

struct Meeting {  // of the lanes of a wave, or of the block
  int live = 0, arrived = 0, gen = 0;
};
struct Wave : Meeting {
  uint64_t v[2][kLanes];
};
struct Fiber {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  bool done = false;
};

inline std::vector<Fiber> fibers;
inline std::vector<Wave> waves;
inline Meeting block;
inline ucontext_t scheduler;
inline std::function<void()> body;
inline int current = 0;
inline dim3 block_idx, block_dim, grid_dim;

inline void yield() { swapcontext(&fibers[current].ctx, &scheduler); }

inline void meet(Meeting& m) {
  const int g = m.gen;
  if (++m.arrived == m.live) {
    m.arrived = 0;
    ++m.gen;
  } else {
    while (m.gen == g) yield();
  }
}

// What every lane of the wave gave; valid until the wave meets twice more.
inline const uint64_t* exchange(uint64_t v) {
  Wave& w = waves[current / kLanes];
  uint64_t* const buf = w.v[w.gen & 1];
  buf[current % kLanes] = v;
  meet(w);
  return buf;
}

inline void leave(Meeting& m) {
  if (--m.live > 0 && m.arrived == m.live) {
    m.arrived = 0;
    ++m.gen;
  }
}

inline void entry() {
  body();
  Fiber& f = fibers[current];
  f.done = true;
  leave(waves[current / kLanes]);
  leave(block);
  yield();
}

// Runs block b of a grid of `blocks` with `threads` (a multiple of 64) each.
inline void run_block(int b, int blocks, int threads, std::function<void()> f) {
  constexpr size_t kStack = 64 * 1024;
  block_idx = dim3(b);
  block_dim = dim3(threads);
  grid_dim = dim3(blocks);
  body = std::move(f);
  fibers = std::vector<Fiber>(threads);
  waves = std::vector<Wave>(threads / kLanes);
  for (Wave& w : waves) w.live = kLanes;
  block = Meeting();
  block.live = threads;
  for (Fiber& fb : fibers) {
    fb.stack.reset(new char[kStack]);
    getcontext(&fb.ctx);
    fb.ctx.uc_stack.ss_sp = fb.stack.get();
    fb.ctx.uc_stack.ss_size = kStack;
    fb.ctx.uc_link = nullptr;
    makecontext(&fb.ctx, entry, 0);
  }
  for (bool left = true; left;) {
    left = false;
    for (current = 0; current < threads; ++current) {
      if (fibers[current].done) continue;
      left = true;
      swapcontext(&scheduler, &fibers[current].ctx);
    }
  }
}

struct Index {
  const bool thread;
  operator unsigned() const { return thread ? (unsigned)current : block_idx.x; }
};
struct Coord { Index x; };

// v_mov_b32 with a DPP control: lane `l`'s source, or -1.
inline int dpp_source(int l, int ctrl) {
  const int r = l & 15, row = l & ~15;
  if (ctrl <= 0xff) return (l & ~3) + (ctrl >> (2 * (l & 3)) & 3);
  if (ctrl > 0x110 && ctrl <= 0x11f) return r >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
  if (ctrl > 0x120 && ctrl <= 0x12f) return row + ((r - (ctrl - 0x120)) & 15);
  if (ctrl == 0x140) return row + 15 - r;
  if (ctrl == 0x141) return (l & ~7) + 7 - (l & 7);
  if (ctrl == 0x142) return row > 0 ? row - 1 : -1;  // last lane of the row before
  if (ctrl == 0x143) return l >= 32 ? 31 : -1;
  if (ctrl >= 0x150 && ctrl <= 0x15f) return row + (ctrl - 0x150);
  __builtin_trap();
}
inline int update_dpp(int old, int src, int ctrl, int rows, int banks) {
  const int l = current % kLanes;
  const uint64_t* const v = exchange((uint32_t)src);
  const int s = dpp_source(l, ctrl);
  const bool on = (rows >> (l / 16) & 1) && (banks >> (l % 16 / 4) & 1);
  return on && s >= 0 ? (int)(uint32_t)v[s] : old;
}
template <typename T>
inline T bits(uint64_t v) {
  T t;
  __builtin_memcpy(&t, &v, sizeof t);
  return t;
}

}  // namespace hip_host

inline const hip_host::Coord threadIdx{{true}}, blockIdx{{false}};
#define blockDim hip_host::block_dim
#define gridDim hip_host::grid_dim

inline void __syncthreads() { hip_host::meet(hip_host::block); }
inline int __lane_id() { return hip_host::current % hip_host::kLanes; }
inline uint64_t __ballot(bool p) {
  const uint64_t* const v = hip_host::exchange(p);
  uint64_t m = 0;
  for (int l = 0; l < hip_host::kLanes; ++l) m |= (v[l] & 1) << l;
  return m;
}
inline int __shfl_up(int v, int n) {
  const int l = __lane_id();
  const uint64_t* const a = hip_host::exchange((uint32_t)v);
  return (int)(uint32_t)a[l >= n ? l - n : l];
}
inline int __shfl_xor(int v, int n) {
  return (int)(uint32_t)hip_host::exchange((uint32_t)v)[__lane_id() ^ n];
}
inline int atomicAdd(int* p, int v) {
  const int old = *p;
  *p += v;
  return old;
}
inline float __uint_as_float(uint32_t u) { return hip_host::bits<float>(u); }
inline float __int_as_float(int u) { return hip_host::bits<float>((uint32_t)u); }
inline uint32_t __float_as_uint(float f) { uint32_t u; __builtin_memcpy(&u, &f, 4); return u; }
inline int __float_as_int(float f) { return (int)__float_as_uint(f); }

#define __builtin_amdgcn_update_dpp(old, src, ctrl, rows, banks, zero) \
  hip_host::update_dpp(old, src, ctrl, rows, banks)
#define __builtin_amdgcn_readlane(v, l) ((int)(uint32_t)hip_host::exchange((uint32_t)(v))[l])
#define __builtin_amdgcn_readfirstlane(v) __builtin_amdgcn_readlane(v, 0)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_sqrtf(x) sqrtf(x)
#define __builtin_amdgcn_s_barrier() __syncthreads()
#define __builtin_amdgcn_make_buffer_rsrc(...) 0
#define __amdgpu_buffer_rsrc_t int
