// Host emulation of the device operations that the kernels' sources use, so
// that tests can compile a .hip file with g++ and run its kernels on the CPU.
//
// A workgroup runs on one host thread, its work-items as fibers: a wavefront
// runs until all its lanes wait for each other (ballot, shuffle, readlane,
// DPP) or for the workgroup's barrier.  Between two barriers the wavefronts
// run one after another in an order drawn from emu::seed, so that an access
// that needs a barrier which is not there shows in some order; a lane that
// sleeps in a polling loop lets the other wavefronts go on.  The
// workgroups of a cooperative launch run side by side, those of an ordinary
// one after another.  Arithmetic wraps (built with -fwrapv).
#pragma once

#include <stdint.h>
#include <sys/mman.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <numeric>
#include <random>
#include <thread>
#include <type_traits>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __shared__ static thread_local

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
using hipStream_t = void*;
using hipError_t = int;
constexpr hipError_t hipSuccess = 0, hipErrorUnknown = 999;
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeWallClockRate };
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  return *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000, hipSuccess;
}
template <typename F>
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, F, int, size_t) {
  return *n = 1, hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }

extern "C" void emu_switch(void** save, void* load);
#ifdef EMU_MAIN
asm(R"(
.text
.globl emu_switch
.type emu_switch,@function
emu_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");
#endif

struct EmuIndex {
  unsigned x = 0, y = 0, z = 0;
};
inline thread_local EmuIndex threadIdx, blockIdx;
inline thread_local dim3 gridDim, blockDim;

namespace emu {

constexpr int kLanes = 64;
constexpr size_t kStack = 64 * 1024;

enum State { kRun, kWaveOp, kBarrier, kSpin, kDone };

struct Fiber {
  void* sp = nullptr;
  State state = kRun;
  int site = 0;  // source line of the wavefront operation it waits in
  uint64_t value = 0;
};

struct Group {  // a workgroup
  std::vector<Fiber> fibers;
  char* stacks = nullptr;
  void* main_sp = nullptr;
  int cur = 0;
  int barrier_or = 0, barrier_result = 0;
  uint64_t snap[kLanes];  // what the active lanes of the running wavefront posted
  uint64_t mask = 0;
  bool spinning = false;
  const std::function<void()>* body = nullptr;
};
inline thread_local Group* g_group = nullptr;
inline uint64_t seed = 0;

[[noreturn]] inline void fail(const char* what) {
  std::fprintf(stderr, "emu: %s\n", what);
  std::abort();
}

inline void yield_to_main(State s) {
  Group& g = *g_group;
  Fiber& f = g.fibers[g.cur];
  f.state = s;
  emu_switch(&f.sp, g.main_sp);
}

inline void entry() {
  (*g_group->body)();
  yield_to_main(kDone);
  fail("a finished work-item was resumed");
}

// Posts x with the wavefront's other active lanes; afterwards snap and mask
// hold what all of them posted.
inline void post(uint64_t x, int line) {
  Group& g = *g_group;
  Fiber& f = g.fibers[g.cur];
  f.value = x;
  f.site = line;
  yield_to_main(kWaveOp);
}

inline void run_wave(Group& g, int first, int last) {
  while (true) {
    for (int i = first; i < last; ++i) {
      Fiber& f = g.fibers[i];
      if (f.state != kRun) continue;
      g.cur = i;
      threadIdx.x = static_cast<unsigned>(i);
      emu_switch(&g.main_sp, f.sp);
    }
    bool spin = false;  // the lanes meet again behind a polling loop
    for (int i = first; i < last; ++i) {
      if (g.fibers[i].state != kSpin) continue;
      g.fibers[i].state = kRun;
      spin = g.spinning = true;
    }
    if (spin) return;
    g.mask = 0;
    int site = 0;
    for (int i = first; i < last; ++i) {
      Fiber& f = g.fibers[i];
      if (f.state != kWaveOp) continue;
      if (site && f.site != site) fail("lanes of a wavefront wait in different operations");
      site = f.site;
      g.mask |= 1ull << (i - first);
      g.snap[i - first] = f.value;
      f.state = kRun;
    }
    if (!g.mask) return;
  }
}

inline void run_group(dim3 grid, dim3 block, unsigned index, const std::function<void()>& body) {
  Group g;
  const int n = static_cast<int>(block.x);
  g.fibers.resize(n);
  g.stacks = static_cast<char*>(mmap(nullptr, kStack * n, PROT_READ | PROT_WRITE,
                                     MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
  if (g.stacks == MAP_FAILED) fail("no memory for stacks");
  g.body = &body;
  g_group = &g;
  gridDim = grid;
  blockDim = block;
  blockIdx.x = index % grid.x;
  blockIdx.y = index / grid.x;
  for (int i = 0; i < n; ++i) {
    // a frame for emu_switch to return into entry() from, the stack aligned as after a call
    void** top = reinterpret_cast<void**>(g.stacks + kStack * (i + 1) - 16);
    *--top = nullptr;
    *--top = reinterpret_cast<void*>(entry);
    for (int r = 0; r < 6; ++r) *--top = nullptr;
    g.fibers[i].sp = top;
  }
  std::mt19937_64 rng(seed * 1000003u + index);
  const int waves = (n + kLanes - 1) / kLanes;
  std::vector<int> order(waves);
  std::iota(order.begin(), order.end(), 0);
  while (true) {
    if (seed) std::shuffle(order.begin(), order.end(), rng);
    for (int w : order) run_wave(g, w * kLanes, std::min(n, (w + 1) * kLanes));
    if (g.spinning) {  // not all at the barrier yet
      g.spinning = false;
      std::this_thread::yield();
      continue;
    }
    bool live = false;
    for (Fiber& f : g.fibers) {
      if (f.state == kBarrier) {
        f.state = kRun;
        live = true;
      }
    }
    g.barrier_result = g.barrier_or;
    g.barrier_or = 0;
    if (!live) break;
  }
  munmap(g.stacks, kStack * n);
  g_group = nullptr;
}

inline void launch(dim3 grid, dim3 block, const std::function<void()>& body, bool together = false) {
  const unsigned blocks = grid.x * grid.y;
  if (!together) {
    for (unsigned i = 0; i < blocks; ++i) run_group(grid, block, i, body);
    return;
  }
  std::vector<std::thread> t;
  for (unsigned i = 0; i < blocks; ++i) t.emplace_back([&, i] { run_group(grid, block, i, body); });
  for (std::thread& x : t) x.join();
}

// Kernels that can be launched through their address (cooperative launches).
using Unpack = std::function<void(void**)>;
inline std::map<const void*, Unpack>& kernels() {
  static std::map<const void*, Unpack> k;
  return k;
}
template <typename... A, size_t... I>
void call(void (*f)(A...), void** a, std::index_sequence<I...>) {
  f(*static_cast<std::remove_reference_t<A>*>(a[I])...);
}
template <typename... A>
void add_kernel(void (*f)(A...)) {
  kernels()[reinterpret_cast<const void*>(f)] = [f](void** a) { call(f, a, std::index_sequence_for<A...>()); };
}

template <typename T>
uint64_t bits(T x) {
  uint64_t u = 0;
  std::memcpy(&u, &x, sizeof(T));
  return u;
}
template <typename T>
T from_bits(uint64_t u) {
  T x;
  std::memcpy(&x, &u, sizeof(T));
  return x;
}
inline int lane() { return static_cast<int>(threadIdx.x) % kLanes; }
// What the lane posted; of a lane outside the operation the value is
// undefined on the device: the caller's own here.
template <typename T>
T of_lane(int l, T own) {
  const Group& g = *g_group;
  return l >= 0 && l < kLanes && (g.mask >> l & 1u) ? from_bits<T>(g.snap[l]) : own;
}

}  // namespace emu

inline hipError_t hipLaunchCooperativeKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  auto it = emu::kernels().find(f);
  if (it == emu::kernels().end()) return hipErrorUnknown;
  emu::launch(grid, block, [&] { it->second(args); }, true);
  return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, shared, stream, ...) \
  emu::launch(grid, block, [&] { (kernel)(__VA_ARGS__); })

#define EMU_LINE int line = __builtin_LINE()
inline int __lane_id() { return emu::lane(); }
inline void __syncthreads() { emu::yield_to_main(emu::kBarrier); }
inline int __syncthreads_or(int x) {
  emu::g_group->barrier_or |= x != 0;
  emu::yield_to_main(emu::kBarrier);
  return emu::g_group->barrier_result;
}
inline uint64_t __ballot(int p, EMU_LINE) {
  emu::post(p ? 1u : 0u, line);
  uint64_t m = 0;
  for (int l = 0; l < emu::kLanes; ++l)
    if ((emu::g_group->mask >> l & 1u) && emu::g_group->snap[l]) m |= 1ull << l;
  return m;
}
template <typename T>
T __shfl(T x, int src, int width = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::of_lane((emu::lane() & ~(width - 1)) + (src & (width - 1)), x);
}
template <typename T>
T __shfl_xor(T x, int m, int = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::of_lane(emu::lane() ^ m, x);
}
template <typename T>
T __shfl_up(T x, int d, int width = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  const int l = emu::lane();
  return (l & (width - 1)) >= d ? emu::of_lane(l - d, x) : x;
}
inline int emu_readlane(int x, int l, EMU_LINE) {
  emu::post(emu::bits(x), line);
  if (!(emu::g_group->mask >> l & 1u)) emu::fail("readlane of an inactive lane");
  return emu::from_bits<int>(emu::g_group->snap[l]);
}
inline int emu_readfirstlane(int x, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::from_bits<int>(emu::g_group->snap[__builtin_ctzll(emu::g_group->mask)]);
}
inline int emu_dpp(int old, int x, int ctrl, int row_mask, bool zero, EMU_LINE) {
  emu::post(emu::bits(x), line);
  const int l = emu::lane(), row = l / 16;
  if (!(row_mask >> row & 1)) return old;
  int src = -1;
  if (ctrl < 0x100) src = (l & ~3) + (ctrl >> (2 * (l & 3)) & 3);
  else if (ctrl > 0x110 && ctrl < 0x120) src = (l & 15) >= (ctrl & 15) ? l - (ctrl & 15) : -1;
  else if (ctrl == 0x140) src = row * 16 + 15 - (l & 15);
  else if (ctrl == 0x141) src = (l & ~7) + 7 - (l & 7);
  else if (ctrl == 0x142) src = row > 0 ? row * 16 - 1 : -1;
  else if (ctrl == 0x143) src = row > 1 ? 31 : -1;
  else emu::fail("DPP control word");
  if (src < 0 || !(emu::g_group->mask >> src & 1u)) return zero ? 0 : old;
  return emu::from_bits<int>(emu::g_group->snap[src]);
}
#define __builtin_amdgcn_readlane(x, l) emu_readlane(x, l)
#define __builtin_amdgcn_readfirstlane(x) emu_readfirstlane(static_cast<int>(x))
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rm, bm, zero) emu_dpp(old, x, ctrl, rm, zero)
#define __builtin_amdgcn_mov_dpp(x, ctrl, rm, bm, zero) emu_dpp(0, x, ctrl, rm, zero)
#define __builtin_amdgcn_mbcnt_lo(m, add) \
  (__builtin_popcount((m) & (emu::lane() >= 32 ? ~0u : (1u << emu::lane()) - 1u)) + (add))
#define __builtin_amdgcn_mbcnt_hi(m, add) \
  (__builtin_popcount((m) & (emu::lane() <= 32 ? 0u : (1u << (emu::lane() - 32)) - 1u)) + (add))
// lanes hand data to each other through LDS here: every lane has to arrive
#define __builtin_amdgcn_wave_barrier() emu::post(0, __LINE__)
#define __builtin_amdgcn_fence(order, scope) __atomic_thread_fence(__ATOMIC_SEQ_CST)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_s_sleep(x) emu::yield_to_main(emu::kSpin)
inline void __threadfence() { __atomic_thread_fence(__ATOMIC_SEQ_CST); }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline long long wall_clock64() {  // 100 MHz
  return std::chrono::steady_clock::now().time_since_epoch() / std::chrono::nanoseconds(10);
}

#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_exchange(p, v, order, scope) __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
template <typename T>
T atomicAdd(T* p, std::common_type_t<T> v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
template <typename T>
T atomicOr(T* p, std::common_type_t<T> v) { return __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }
template <typename T>
T atomicAnd(T* p, std::common_type_t<T> v) { return __atomic_fetch_and(p, v, __ATOMIC_SEQ_CST); }
template <typename T>
T atomicExch(T* p, std::common_type_t<T> v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
template <typename T>
T atomicCAS(T* p, std::common_type_t<T> cmp, std::common_type_t<T> v) {
  __atomic_compare_exchange_n(p, &cmp, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return cmp;
}
template <typename T>
T atomicMax(T* p, std::common_type_t<T> v) {
  T old = *p;
  while (old < v && !__atomic_compare_exchange_n(p, &old, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {}
  return old;
}
template <typename T>
T atomicMin(T* p, std::common_type_t<T> v) {
  T old = *p;
  while (v < old && !__atomic_compare_exchange_n(p, &old, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {}
  return old;
}
using std::max;
using std::min;
