// Stand-in for the HIP device runtime that lets g++ build scan.hpp: a
// workgroup is a set of contexts (64 per wave) that one host thread switches
// between, the wave and workgroup operations are barriers around shared
// arrays, global atomics are the host's.  Only what scan.hpp uses.
#pragma once

#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <thread>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __builtin_amdgcn_s_sleep(n) cpu::group->yield()

namespace cpu {

struct Dim3 {
  unsigned x = 0;
};
inline thread_local Dim3 thread_idx, block_idx;

struct Group {
  struct Barrier {
    int want = 0, arrived = 0;
    unsigned round = 0;
  };
  struct Wave {
    Barrier bar;
    uint64_t slot[64];
  };
  struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    bool done = false;
  };
  explicit Group(int n) : flag(n), waves(n / 64), lanes(n) {
    all.want = n;
    for (auto& w : waves) w.bar.want = 64;
  }
  void yield() { swapcontext(&lanes[thread_idx.x].ctx, &home); }
  void wait(Barrier& b) {
    const unsigned round = b.round;
    if (++b.arrived == b.want) {
      b.arrived = 0;
      ++b.round;
    } else {
      while (b.round == round) yield();
    }
  }
  Barrier all;
  std::vector<int> flag;
  std::vector<Wave> waves;
  std::vector<Lane> lanes;
  ucontext_t home;
  const std::function<void()>* body = nullptr;
};
inline thread_local Group* group = nullptr;

inline void lane_main() {
  (*group->body)();
  group->lanes[thread_idx.x].done = true;
  group->yield();
}

// Runs f as workgroup `block` of `threads` threads (a multiple of 64).
inline void run_block(unsigned block, int threads, const std::function<void()>& f) {
  Group g(threads);
  g.body = &f;
  group = &g;
  block_idx.x = block;
  for (auto& l : g.lanes) {
    l.stack.resize(1 << 16);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.data();
    l.ctx.uc_stack.ss_size = l.stack.size();
    l.ctx.uc_link = nullptr;
    makecontext(&l.ctx, lane_main, 0);
  }
  for (int left = threads; left > 0;) {
    left = 0;
    for (int t = 0; t < threads; ++t) {
      if (g.lanes[t].done) continue;
      thread_idx.x = static_cast<unsigned>(t);
      swapcontext(&g.home, &g.lanes[t].ctx);
      left += g.lanes[t].done ? 0 : 1;
    }
  }
}

inline Group::Wave& wave() { return group->waves[thread_idx.x >> 6]; }

// this wave's 64 values of v, seen by `pick`
template <typename T, typename F>
inline auto exchange(T v, F pick) {
  Group::Wave& w = wave();
  uint64_t bits = 0;
  memcpy(&bits, &v, sizeof(T));
  w.slot[thread_idx.x & 63] = bits;
  group->wait(w.bar);
  auto r = pick(w.slot);
  group->wait(w.bar);
  return r;
}

template <typename T>
inline T lane_value(const uint64_t* slot, int lane) {
  T v;
  memcpy(&v, &slot[lane], sizeof(T));
  return v;
}

}  // namespace cpu

#define threadIdx cpu::thread_idx
#define blockIdx cpu::block_idx

inline void __syncthreads() { cpu::group->wait(cpu::group->all); }
inline int __syncthreads_and(int p) {
  cpu::Group& g = *cpu::group;
  g.flag[threadIdx.x] = p;
  g.wait(g.all);
  int r = 1;
  for (int f : g.flag) r &= f != 0;
  g.wait(g.all);
  return r;
}
template <typename T>
inline T __shfl_up(T v, int delta, int) {
  const int lane = threadIdx.x & 63;
  return cpu::exchange(v, [=](const uint64_t* s) { return cpu::lane_value<T>(s, lane >= delta ? lane - delta : lane); });
}
template <typename T>
inline T __shfl_xor(T v, int mask, int) {
  const int lane = threadIdx.x & 63;
  return cpu::exchange(v, [=](const uint64_t* s) { return cpu::lane_value<T>(s, lane ^ mask); });
}
inline uint64_t __ballot(int p) {
  return cpu::exchange<uint64_t>(p != 0, [](const uint64_t* s) {
    uint64_t m = 0;
    for (int i = 0; i < 64; ++i) m |= (s[i] & 1) << i;
    return m;
  });
}
inline int __any(int p) { return __ballot(p) != 0; }
inline int __ffsll(long long x) { return __builtin_ffsll(x); }
inline uint32_t atomicAdd(uint32_t* p, uint32_t v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
