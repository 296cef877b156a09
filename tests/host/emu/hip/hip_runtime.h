// Stands in for the HIP runtime header where a host check compiles kernels of the library as plain C++
// and runs them on the CPU: every GPU thread is a fiber, the fibers of a wave advance together from
// one meeting point (barrier, exchange between lanes) to the next, and the order in which the waves of a
// launch get their turns is the check's choice -- so an order that the hardware takes once in a
// million launches can be asked for.  Memory is the host's: an out-of-range access is the sanitizer's to
// find.  Covers what the files under check use, no more.
#pragma once
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <random>
#include <vector>

#undef __global__
#undef __device__
#undef __host__
#undef __forceinline__
#undef __launch_bounds__
#undef __shared__
#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static  // one workgroup at a time: only under Order::kByGroup

using std::max;
using std::min;

namespace emu {

constexpr int kWave = 64;
constexpr size_t kStack = 64 << 10;

// Which (workgroup, wave) goes on next, of those that can.
enum class Order {
  kByGroup,       // one workgroup after the other
  kLeadersFirst,  // wave 0 of every workgroup, then wave 1 of every workgroup, ...
  kLeadersLast,   // the last waves first
  kRandom,
};
inline Order order = Order::kByGroup;
inline std::mt19937 rng(1);

enum State { kReady, kAtBarrier, kAtExchange, kDone };
struct Thread {
  ucontext_t context;
  unsigned char *stack = nullptr;
  State state = kReady;
  dim3 thread, block;
  int group = 0;
  unsigned exchanges = 0;                 // how many exchanges the thread has taken part in
  unsigned long long published[2] = {};   // its value of the last two
};
inline std::vector<Thread> threads;
inline int per_group = 0, now = -1;
inline ucontext_t scheduler;
inline std::function<void()> body;
inline dim3 grid_dim, block_dim;

inline void leave(State s) {
  Thread &t = threads[now];
  t.state = s;
  swapcontext(&t.context, &scheduler);
}
inline void entry() {
  body();
  leave(kDone);
}
inline int lane() { return (int)(threads[now].thread.x % kWave); }
// The values of all lanes of the wave (of a thread beyond the workgroup's end: 0).
struct WaveValues {
  unsigned long long v[kWave];
};
inline WaveValues exchange(unsigned long long mine) {
  const int me = now;
  const unsigned turn = threads[me].exchanges++ & 1;
  threads[me].published[turn] = mine;
  leave(kAtExchange);
  WaveValues w;
  const int first = me - lane(), end = (threads[me].group + 1) * per_group;
  for (int i = 0; i < kWave; ++i) w.v[i] = first + i < end ? threads[first + i].published[turn] : 0;
  return w;
}

inline void launch(dim3 grid, dim3 block, std::function<void()> fn) {
  const int groups = (int)(grid.x * grid.y * grid.z), waves = ((int)block.x + kWave - 1) / kWave;
  per_group = (int)block.x;
  grid_dim = grid;
  block_dim = block;
  body = std::move(fn);
  threads.assign((size_t)groups * per_group, Thread());
  const size_t bytes = threads.size() * kStack;
  unsigned char *const stacks =
      (unsigned char *)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (stacks == MAP_FAILED) abort();
  for (size_t i = 0; i < threads.size(); ++i) {
    Thread &t = threads[i];
    t.group = (int)(i / per_group);
    t.thread = dim3((unsigned)(i % per_group), 0, 0);
    t.block = dim3(t.group % grid.x, t.group / grid.x % grid.y, t.group / (grid.x * grid.y));
    t.stack = stacks + i * kStack;
    getcontext(&t.context);
    t.context.uc_stack.ss_sp = t.stack;
    t.context.uc_stack.ss_size = kStack;
    t.context.uc_link = nullptr;
    makecontext(&t.context, entry, 0);
  }
  std::vector<int> units;  // group * waves + wave, those that have not ended
  for (int u = 0; u < groups * waves; ++u) units.push_back(u);
  auto range = [&](int u, int &a, int &b) {
    a = u / waves * per_group + u % waves * kWave;
    b = min(a + kWave, (u / waves + 1) * per_group);
  };
  auto any = [&](int a, int b, State s) {
    for (int i = a; i < b; ++i)
      if (threads[i].state == s) return true;
    return false;
  };
  if (order == Order::kLeadersFirst || order == Order::kLeadersLast)
    std::stable_sort(units.begin(), units.end(), [&](int x, int y) {
      return order == Order::kLeadersFirst ? x % waves < y % waves : x % waves > y % waves;
    });
  while (!units.empty()) {
    std::vector<int> can;
    for (int u : units) {
      int a, b;
      range(u, a, b);
      if (any(a, b, kReady)) {
        can.push_back(u);
        if (order != Order::kRandom) break;
      }
    }
    if (can.empty()) {
      printf("FAILED: every wave waits\n");
      exit(1);
    }
    const int u = can[rng() % can.size()];
    int a, b;
    range(u, a, b);
    while (any(a, b, kReady)) {  // to the wave's next barrier, or its end
      for (now = a; now < b; ++now)
        if (threads[now].state == kReady) {
          const int i = now;
          swapcontext(&scheduler, &threads[i].context);
          now = i;
        }
      if (any(a, b, kAtExchange) && !any(a, b, kAtBarrier) && !any(a, b, kDone))
        for (int i = a; i < b; ++i) threads[i].state = kReady;
    }
    if (any(a, b, kAtExchange)) {
      printf("FAILED: an exchange that not all lanes take part in\n");
      exit(1);
    }
    const int ga = u / waves * per_group, gb = ga + per_group;
    if (any(ga, gb, kAtBarrier) && !any(ga, gb, kReady) && !any(ga, gb, kAtExchange))
      for (int i = ga; i < gb; ++i)
        if (threads[i].state == kAtBarrier) threads[i].state = kReady;
    if (!any(a, b, kReady) && !any(a, b, kAtBarrier)) units.erase(std::find(units.begin(), units.end(), u));
  }
  now = -1;
  munmap(stacks, bytes);
}

}  // namespace emu

#define threadIdx (emu::threads[emu::now].thread)
#define blockIdx (emu::threads[emu::now].block)
#define gridDim (emu::grid_dim)
#define blockDim (emu::block_dim)
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
  emu::launch((grid), (block), [&] { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { emu::leave(emu::kAtBarrier); }
template <typename T>
inline T atomicAdd(T *at, T x) {
  emu::leave(emu::kReady);  // the wave's other lanes come as far as this one first
  const T old = *at;
  *at = old + x;
  return old;
}
inline float __uint_as_float(unsigned x) { return __builtin_bit_cast(float, x); }
inline unsigned __float_as_uint(float x) { return __builtin_bit_cast(unsigned, x); }

// exchanges between the lanes of a wave
inline unsigned long long emu_ballot(bool x) {
  const emu::WaveValues w = emu::exchange(x);
  unsigned long long m = 0;
  for (int i = 0; i < emu::kWave; ++i) m |= (w.v[i] & 1ull) << i;
  return m;
}
inline int emu_readlane(int x, int from) { return (int)emu::exchange((unsigned)x).v[from]; }
inline int emu_readfirstlane(int x) { return emu_readlane(x, 0); }
inline int emu_dpp(int x, int control) {
  const emu::WaveValues w = emu::exchange((unsigned)x);
  const int l = emu::lane(), row = l & ~15, in_row = l & 15;
  switch (control) {
    case 0xB1: return (int)w.v[l ^ 1];                     // quad_perm [1,0,3,2]
    case 0x4E: return (int)w.v[l ^ 2];                     // quad_perm [2,3,0,1]
    case 0x141: return (int)w.v[(l & ~7) | (7 - (l & 7))];  // row_half_mirror
    case 0x140: return (int)w.v[row | (15 - in_row)];      // row_mirror
  }
  printf("FAILED: unknown lane exchange %x\n", control);
  exit(1);
}
inline unsigned emu_mbcnt(unsigned mask, unsigned add, int first) {
  const int l = emu::lane() - first;
  const unsigned below = l <= 0 ? 0u : l >= 32 ? ~0u : (1u << l) - 1u;
  return add + (unsigned)__builtin_popcount(mask & below);
}
#define __builtin_amdgcn_s_barrier() __syncthreads()
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(at, order, scope) (*(at))
#define __hip_atomic_store(at, x, order, scope) (*(at) = (x))
#define __builtin_amdgcn_s_waitcnt(counts) ((void)0)  // a fiber has what it has loaded
#define __builtin_amdgcn_ballot_w64(x) emu_ballot(x)
#define __builtin_amdgcn_readlane(x, from) emu_readlane((x), (from))
#define __builtin_amdgcn_readfirstlane(x) emu_readfirstlane(x)
#define __builtin_amdgcn_mov_dpp(x, control, rows, banks, bound) emu_dpp((x), (control))
#define __builtin_amdgcn_mbcnt_lo(mask, add) emu_mbcnt((mask), (add), 0)
#define __builtin_amdgcn_mbcnt_hi(mask, add) emu_mbcnt((mask), (add), 32)
