// One thread block of a kernel on the CPU: every thread is a fibre, and the
// wavefront and block operations that the kernels use are rendezvous points.
// A block barrier ends only when every thread of the block stands at it: one
// that some threads reach at another line, where the hardware would pair two
// different barriers, is reported.  Included in place of the HIP header when
// a kernel's source is compiled for the host; only what those sources use.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <string>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static  // one block at a time

typedef int hipError_t;
typedef void* hipStream_t;

struct float2 {
  float x, y;
};

namespace cpu {

struct Idx {
  unsigned x, y, z;
};

struct Fibre {
  ucontext_t at;
  std::vector<char> stack;
  bool done, waits;
  int line;  // of the operation it waits at
  uint64_t value;
};

struct Block {
  std::vector<Fibre> f;
  std::vector<std::vector<uint64_t>> seen;  // [wavefront] the last rendezvous' values
  ucontext_t home;
  int cur = 0;
  std::string fault;
  std::function<void()> body;
};

inline Block* blk;
inline Idx block_idx;
// Called for every agent-scope load of a flag: (address, wavefront) -> value.
inline std::function<float(const float*, int)> on_load;

inline void yield() { swapcontext(&blk->f[blk->cur].at, &blk->home); }

// All 64 lanes of the wavefront leave a value at `line`; returns the values.
inline const std::vector<uint64_t>& meet(uint64_t value, int line) {
  Fibre& me = blk->f[blk->cur];
  me.value = value;
  me.line = line;
  me.waits = true;
  yield();
  return blk->seen[blk->cur / 64];
}

// Block barriers have negative lines.
inline void barrier(int line) {
  Fibre& me = blk->f[blk->cur];
  me.line = -line;
  me.waits = true;
  yield();
}

inline void entry() {
  blk->body();
  blk->f[blk->cur].done = true;
  yield();
}

// Runs the block; "" or the fault that ended it.
inline std::string run(int threads, unsigned x, std::function<void()> body) {
  Block b;
  blk = &b;
  block_idx = Idx{x, 0, 0};
  b.body = body;
  b.f.resize(threads);
  b.seen.assign(threads / 64, std::vector<uint64_t>(64));
  for (auto& f : b.f) {
    f.stack.resize(64 << 10);
    f.done = f.waits = false;
    getcontext(&f.at);
    f.at.uc_stack.ss_sp = f.stack.data();
    f.at.uc_stack.ss_size = f.stack.size();
    f.at.uc_link = nullptr;
    makecontext(&f.at, entry, 0);
  }
  while (b.fault.empty()) {
    int live = 0, moved = 0;
    for (int v = 0; v < threads / 64; ++v) {
      // each lane of the wavefront to its next rendezvous or its end
      for (int l = 64 * v; l < 64 * v + 64; ++l) {
        Fibre& f = b.f[l];
        if (f.done) continue;
        if (!f.waits) {
          b.cur = l;
          swapcontext(&b.home, &f.at);
          ++moved;
        }
        live += !f.done;
      }
      const Fibre& f0 = b.f[64 * v];
      for (int l = 64 * v; l < 64 * v + 64; ++l)
        if (b.f[l].done != f0.done || (!f0.done && b.f[l].line != f0.line)) b.fault = "lanes of a wavefront part";
      if (!f0.done && f0.line > 0)
        for (int l = 0; l < 64; ++l) {
          b.seen[v][l] = b.f[64 * v + l].value;
          b.f[64 * v + l].waits = false;
        }
    }
    if (!live) break;
    if (moved) continue;
    // every live wavefront waits at a block barrier
    int line = 0;
    for (auto& f : b.f)
      if (!f.done) {
        if (line && f.line != line)
          b.fault = "wavefronts wait at block barriers of lines " + std::to_string(-line) + " and " + std::to_string(-f.line);
        line = f.line;
        f.waits = false;
      }
  }
  blk = nullptr;
  return b.fault;
}

inline int lane() { return blk->cur & 63; }

inline uint64_t ballot(bool p, int line) {
  const auto& s = meet(p, line);
  uint64_t r = 0;
  for (int l = 0; l < 64; ++l) r |= (s[l] & 1) << l;
  return r;
}

// Lane `from`'s 32 bits; 0 for a negative lane.
inline uint32_t lane32(uint32_t x, int from, int line) {
  const auto& s = meet(x, line);
  return from < 0 ? 0u : (uint32_t)s[from];
}

template <typename T>
inline T lane_any(T x, int from, int line) {
  uint64_t u = 0;
  memcpy(&u, &x, sizeof x);
  const uint64_t y = meet(u, line)[from];
  memcpy(&x, &y, sizeof x);
  return x;
}

// The source lane of a DPP control word (row_shr, row_bcast:15 and :31), -1
// where the row mask or the row's edge leaves the old value, 0.
inline int dpp_lane(int ctrl, int rows) {
  const int l = lane(), r = l / 16;
  if (!((rows >> r) & 1)) return -1;
  if (ctrl > 0x110 && ctrl < 0x120) return l % 16 >= (ctrl & 15) ? l - (ctrl & 15) : -1;
  if (ctrl == 0x142) return 16 * r - 1;
  return ctrl == 0x143 && r >= 2 ? 31 : -1;
}

inline int vote(int p, int line, bool count) {
  static int n;
  barrier(line);
  if (blk->cur == 0) n = 0;
  barrier(line);
  n += count || !n ? p != 0 : 0;
  barrier(line);
  return n;
}

}  // namespace cpu

#define threadIdx (cpu::Idx{(unsigned)cpu::blk->cur, 0, 0})
#define blockIdx (cpu::block_idx)
#define blockDim (cpu::Idx{(unsigned)cpu::blk->f.size(), 1, 1})
#define __syncthreads() cpu::barrier(__LINE__)
#define __syncthreads_or(p) cpu::vote(p, __LINE__, false)
#define __syncthreads_count(p) cpu::vote(p, __LINE__, true)
#define __ballot(p) cpu::ballot(p, __LINE__)
#define __all(p) (cpu::ballot(p, __LINE__) == ~0ull)
#define __any(p) (cpu::ballot(p, __LINE__) != 0)
#define __shfl_xor(x, m, w) cpu::lane_any(x, cpu::lane() ^ (m), __LINE__)
#define __builtin_amdgcn_readlane(x, l) (int)cpu::lane32((uint32_t)(x), l, __LINE__)
#define __builtin_amdgcn_readfirstlane(x) (int)cpu::lane32((uint32_t)(x), 0, __LINE__)
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, bound) \
  (int)cpu::lane32((uint32_t)(x), cpu::dpp_lane(ctrl, rows), __LINE__)
#define __builtin_amdgcn_inverse_ballot_w64(m) ((bool)(((m) >> cpu::lane()) & 1))
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)cpu::meet(0, __LINE__))
#define __builtin_nontemporal_load(p) (*(p))
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_load(p, order, scope) cpu::on_load(p, cpu::blk->cur / 64)
#define __hip_atomic_store(p, v, order, scope) ((void)(*(p) = (v)))
#define __popcll(x) __builtin_popcountll(x)

template <typename T, typename U>
inline T atomicOr(T* p, U v) {
  const T o = *p;
  *p |= (T)v;
  return o;
}
template <typename T, typename U>
inline T atomicAdd(T* p, U v) {
  const T o = *p;
  *p += (T)v;
  return o;
}
template <typename T, typename F>
inline T as_bits(F x) {
  T y;
  memcpy(&y, &x, sizeof y);
  return y;
}
inline uint32_t __float_as_uint(float x) { return as_bits<uint32_t>(x); }
inline float __uint_as_float(uint32_t x) { return as_bits<float>(x); }
inline long long __double_as_longlong(double x) { return as_bits<long long>(x); }
inline double __longlong_as_double(long long x) { return as_bits<double>(x); }
