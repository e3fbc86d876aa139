// Host emulation of the device operations that the kernels' sources use, so
// that tests can compile a .hip file with g++ and run its kernels on the CPU.
//
// A workgroup runs on one host thread, its work-items as fibers: a wavefront
// runs until all its lanes wait for each other (ballot, shuffle, readlane,
// DPP) or for the workgroup's barrier.  Between two barriers the wavefronts
// run one after another in an order drawn from emu::seed, so that an access
// that needs a barrier which is not there shows in some order; a lane that
// sleeps in a polling loop lets the other wavefronts go on.  The
// workgroups of a cooperative launch, and of any small one, run side by side,
// else one after another.  Arithmetic wraps (built with -fwrapv).
//
// Host calls work on the one memory there is.  Without emu::start_queues
// everything runs inside the call; with it, streams are spread over so many
// threads (the hardware queues), each in order.
#pragma once

#include <stdint.h>
#include <sys/mman.h>

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <deque>
#include <mutex>
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
using hipStream_t = struct EmuStream*;
using hipEvent_t = struct EmuEvent*;
using hipError_t = int;
constexpr hipError_t hipSuccess = 0, hipErrorNotReady = 600, hipErrorUnknown = 999;
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeWallClockRate };
namespace emu {
inline int cus = 256;
}
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  return *v = a == hipDeviceAttributeMultiprocessorCount ? emu::cus : 100000, hipSuccess;
}
template <typename F>
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, F, int, size_t) {
  return *n = 1, hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }

// Under ThreadSanitizer (-fsanitize=thread) device-scope accesses are atomic
// but order nothing: it then reports every access inside a launch that is
// neither device-scope nor ordered by a barrier of its workgroup.
#ifdef __SANITIZE_THREAD__
#include <sanitizer/tsan_interface.h>
#define EMU_ORDER __ATOMIC_RELAXED
#define EMU_FENCE ((void)0)
#define EMU_TSAN(x) x
#else
#define EMU_ORDER __ATOMIC_SEQ_CST
#define EMU_FENCE __atomic_thread_fence(__ATOMIC_SEQ_CST)
#define EMU_TSAN(x)
#endif

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
  EMU_TSAN(void* tsan = nullptr;)
  State state = kRun;
  int line = 0;                // source line and
  const char* site = nullptr;  // call site of the wavefront operation it waits in
  uint64_t value = 0;
};

struct Group {  // a workgroup
  std::vector<Fiber> fibers;
  char* stacks = nullptr;
  void* main_sp = nullptr;
  EMU_TSAN(void* tsan = nullptr;)
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
  EMU_TSAN(__tsan_switch_to_fiber(g.tsan, 0);)
  emu_switch(&f.sp, g.main_sp);
}

inline void entry() {
  (*g_group->body)();
  yield_to_main(kDone);
  fail("a finished work-item was resumed");
}

// Posts x with the wavefront's other active lanes; afterwards snap and mask
// hold what all of them posted.
__attribute__((noinline)) inline void post(uint64_t x, int line) {
  Group& g = *g_group;
  Fiber& f = g.fibers[g.cur];
  f.value = x;
  f.line = line;
  f.site = static_cast<const char*>(__builtin_return_address(0));
  yield_to_main(kWaveOp);
}

inline void run_wave(Group& g, int first, int last) {
  while (true) {
    for (int i = first; i < last; ++i) {
      Fiber& f = g.fibers[i];
      if (f.state != kRun) continue;
      g.cur = i;
      threadIdx.x = static_cast<unsigned>(i);
      EMU_TSAN(__tsan_switch_to_fiber(f.tsan, 0);)
      emu_switch(&g.main_sp, f.sp);
    }
    bool spin = false;  // the lanes meet again behind a polling loop
    for (int i = first; i < last; ++i) {
      if (g.fibers[i].state != kSpin) continue;
      g.fibers[i].state = kRun;
      spin = g.spinning = true;
    }
    if (spin) return;
    // Lanes that have left a loop or a branch wait for the others where these
    // join them, further on in the code: the operation at the lowest address
    // comes first (built without reordering of blocks).
    const Fiber* at = nullptr;
    for (int i = first; i < last; ++i) {
      const Fiber& f = g.fibers[i];
      if (f.state == kWaveOp && (!at || f.site < at->site)) at = &f;
    }
    g.mask = 0;
    for (int i = first; at && i < last; ++i) {
      Fiber& f = g.fibers[i];
      if (f.state != kWaveOp || f.line != at->line) continue;
      g.mask |= 1ull << (i - first);
      g.snap[i - first] = f.value;
      f.state = kRun;
    }
    if (!g.mask) return;
  }
}

// The stacks of a host thread's workgroup, kept for its next one.
struct Stacks {
  char* p = nullptr;
  int n = 0;
  char* of(int want) {
    if (want > n) {
      drop();
      p = static_cast<char*>(mmap(nullptr, kStack * want, PROT_READ | PROT_WRITE,
                                  MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
      if (p == MAP_FAILED) fail("no memory for stacks");
      n = want;
    }
    return p;
  }
  void drop() {
    if (p) munmap(p, kStack * n);
    p = nullptr;
    n = 0;
  }
#ifdef __SANITIZE_THREAD__
  std::vector<void*> tsan;
  void* fiber(int i) {
    while (static_cast<int>(tsan.size()) <= i) tsan.push_back(__tsan_create_fiber(0));
    return tsan[i];
  }
  ~Stacks() {
    for (void* f : tsan) __tsan_destroy_fiber(f);
    drop();
  }
#else
  ~Stacks() { drop(); }
#endif
};
inline thread_local Stacks t_stacks;

inline void run_group(dim3 grid, dim3 block, unsigned index, const std::function<void()>& body) {
  Group g;
  const int n = static_cast<int>(block.x);
  g.fibers.resize(n);
  g.stacks = t_stacks.of(n);
  EMU_TSAN(g.tsan = __tsan_get_current_fiber();)
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
    EMU_TSAN(g.fibers[i].tsan = t_stacks.fiber(i);)
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
  g_group = nullptr;
}

inline void launch(dim3 grid, dim3 block, const std::function<void()>& body, bool together = false) {
  const unsigned blocks = grid.x * grid.y;
  if (!together && (blocks == 1 || blocks > 16)) {
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

// A hardware queue: work in order, on a thread of its own.
class Queue {
 public:
  Queue() : thread_([this] { run(); }) {}
  ~Queue() {
    push(nullptr);
    thread_.join();
  }
  uint64_t push(std::function<void()> f) {
    std::lock_guard<std::mutex> lk(mu_);
    work_.push_back(std::move(f));
    cv_.notify_all();
    return ++submitted_;
  }
  bool done(uint64_t ticket) {
    std::lock_guard<std::mutex> lk(mu_);
    return done_ >= ticket;
  }
  void wait(uint64_t ticket) {
    std::unique_lock<std::mutex> lk(mu_);
    cv_.wait(lk, [&] { return done_ >= ticket; });
  }
  uint64_t last() {
    std::lock_guard<std::mutex> lk(mu_);
    return submitted_;
  }

 private:
  void run() {
    while (true) {
      std::function<void()> f;
      {
        std::unique_lock<std::mutex> lk(mu_);
        cv_.wait(lk, [&] { return !work_.empty(); });
        f = std::move(work_.front());
        work_.pop_front();
      }
      if (!f) return;
      f();
      std::lock_guard<std::mutex> lk(mu_);
      ++done_;
      cv_.notify_all();
    }
  }
  std::mutex mu_;
  std::condition_variable cv_;
  std::deque<std::function<void()>> work_;
  uint64_t submitted_ = 0, done_ = 0;
  std::thread thread_;
};
inline std::vector<Queue*> queues;
inline std::mutex host_mu;
inline std::map<const char*, size_t> pinned_size;  // pinned host allocations
inline int next_queue = 0;

inline void start_queues(int n) {
  for (int i = 0; i < n; ++i) queues.push_back(new Queue());
}
inline void stop_queues() {
  for (Queue* q : queues) delete q;
  queues.clear();
}
inline bool is_pinned(const void* p) {
  std::lock_guard<std::mutex> lk(host_mu);
  auto it = pinned_size.upper_bound(static_cast<const char*>(p));
  return it != pinned_size.begin() && static_cast<const char*>(p) < (--it)->first + it->second;
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

struct EmuStream {
  emu::Queue* q;
};
struct EmuEvent {
  emu::Queue* q = nullptr;
  uint64_t ticket = 0;
};
namespace emu {
inline Queue* queue_of(hipStream_t s) { return s ? s->q : queues.empty() ? nullptr : queues[0]; }
inline void enqueue(hipStream_t s, std::function<void()> f) {
  if (Queue* q = queue_of(s)) q->push(std::move(f));
  else f();
}
template <typename... P, typename... A>
void enqueue_kernel(void (*k)(P...), dim3 grid, dim3 block, hipStream_t s, A... a) {
  enqueue(s, [=] { launch(grid, block, [&] { k(a...); }); });
}
inline void sync_all() {
  for (Queue* q : queues) q->wait(q->last());
}
}  // namespace emu

enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocDefault = 0;
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = new EmuStream{emu::queues.empty() ? nullptr : emu::queues[emu::next_queue++ % emu::queues.size()]};
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
  if (emu::Queue* q = emu::queue_of(s)) q->wait(q->last());
  return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
  (void)hipStreamSynchronize(s);
  delete s;
  return hipSuccess;
}
inline hipError_t hipEventCreate(hipEvent_t* e) { return *e = new EmuEvent(), hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
inline hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  e->q = emu::queue_of(s);
  if (e->q) e->ticket = e->q->push([] {});
  return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) { return !e->q || e->q->done(e->ticket) ? hipSuccess : hipErrorNotReady; }
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  if (e->q) e->q->wait(e->ticket);
  return hipSuccess;
}
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0, hipSuccess; }
template <typename T>
hipError_t hipMalloc(T** p, size_t n) {
  return *p = static_cast<T*>(std::malloc(n)), *p ? hipSuccess : hipErrorUnknown;
}
inline hipError_t hipFree(void* p) {
  emu::sync_all();
  std::free(p);
  return hipSuccess;
}
template <typename T>
hipError_t hipHostMalloc(T** p, size_t n, unsigned = 0) {
  *p = static_cast<T*>(std::malloc(n));
  std::lock_guard<std::mutex> lk(emu::host_mu);
  emu::pinned_size[reinterpret_cast<const char*>(*p)] = n;
  return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
  emu::sync_all();
  {
    std::lock_guard<std::mutex> lk(emu::host_mu);
    emu::pinned_size.erase(static_cast<const char*>(p));
  }
  std::free(p);
  return hipSuccess;
}
// (a copy from or to pageable host memory is done when the call returns)
inline hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind kind, hipStream_t s) {
  emu::enqueue(s, [=] { std::memcpy(to, from, n); });
  const void* host = kind == hipMemcpyHostToDevice ? from : to;
  if (kind != hipMemcpyDeviceToDevice && !emu::is_pinned(host)) return hipStreamSynchronize(s);
  return hipSuccess;
}
inline hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind kind) {
  (void)hipMemcpyAsync(to, from, n, kind, nullptr);
  return hipStreamSynchronize(nullptr);
}
inline hipError_t hipMemsetAsync(void* p, int x, size_t n, hipStream_t s) {
  emu::enqueue(s, [=] { std::memset(p, x, n); });
  return hipSuccess;
}

inline hipError_t hipLaunchCooperativeKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  auto it = emu::kernels().find(f);
  if (it == emu::kernels().end()) return hipErrorUnknown;
  emu::launch(grid, block, [&] { it->second(args); }, true);
  return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, shared, stream, ...) \
  emu::enqueue_kernel(kernel, grid, block, stream, __VA_ARGS__)

#define EMU_OP inline __attribute__((always_inline))
#define EMU_LINE int line = __builtin_LINE()
inline int __lane_id() { return emu::lane(); }
inline void __syncthreads() { emu::yield_to_main(emu::kBarrier); }
inline int __syncthreads_or(int x) {
  emu::g_group->barrier_or |= x != 0;
  emu::yield_to_main(emu::kBarrier);
  return emu::g_group->barrier_result;
}
EMU_OP uint64_t __ballot(int p, EMU_LINE) {
  emu::post(p ? 1u : 0u, line);
  uint64_t m = 0;
  for (int l = 0; l < emu::kLanes; ++l)
    if ((emu::g_group->mask >> l & 1u) && emu::g_group->snap[l]) m |= 1ull << l;
  return m;
}
template <typename T>
EMU_OP T __shfl(T x, int src, int width = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::of_lane((emu::lane() & ~(width - 1)) + (src & (width - 1)), x);
}
template <typename T>
EMU_OP T __shfl_xor(T x, int m, int = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::of_lane(emu::lane() ^ m, x);
}
template <typename T>
EMU_OP T __shfl_up(T x, int d, int width = 64, EMU_LINE) {
  emu::post(emu::bits(x), line);
  const int l = emu::lane();
  return (l & (width - 1)) >= d ? emu::of_lane(l - d, x) : x;
}
EMU_OP int emu_readlane(int x, int l, EMU_LINE) {
  emu::post(emu::bits(x), line);
  if (!(emu::g_group->mask >> l & 1u)) emu::fail("readlane of an inactive lane");
  return emu::from_bits<int>(emu::g_group->snap[l]);
}
EMU_OP int emu_readfirstlane(int x, EMU_LINE) {
  emu::post(emu::bits(x), line);
  return emu::from_bits<int>(emu::g_group->snap[__builtin_ctzll(emu::g_group->mask)]);
}
EMU_OP int emu_dpp(int old, int x, int ctrl, int row_mask, bool zero, EMU_LINE) {
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
#define __builtin_amdgcn_fence(order, scope) EMU_FENCE
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_s_sleep(x) emu::yield_to_main(emu::kSpin)
inline void __threadfence() { EMU_FENCE; }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline long long wall_clock64() {  // 100 MHz
  return std::chrono::steady_clock::now().time_since_epoch() / std::chrono::nanoseconds(10);
}

#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, EMU_ORDER)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, EMU_ORDER)
#define __hip_atomic_exchange(p, v, order, scope) __atomic_exchange_n(p, v, EMU_ORDER)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, EMU_ORDER)
template <typename T>
T atomicAdd(T* p, std::common_type_t<T> v) { return __atomic_fetch_add(p, v, EMU_ORDER); }
template <typename T>
T atomicOr(T* p, std::common_type_t<T> v) { return __atomic_fetch_or(p, v, EMU_ORDER); }
template <typename T>
T atomicAnd(T* p, std::common_type_t<T> v) { return __atomic_fetch_and(p, v, EMU_ORDER); }
template <typename T>
T atomicExch(T* p, std::common_type_t<T> v) { return __atomic_exchange_n(p, v, EMU_ORDER); }
template <typename T>
T atomicCAS(T* p, std::common_type_t<T> cmp, std::common_type_t<T> v) {
  __atomic_compare_exchange_n(p, &cmp, v, false, EMU_ORDER, EMU_ORDER);
  return cmp;
}
template <typename T>
T atomicMax(T* p, std::common_type_t<T> v) {
  T old = __atomic_load_n(p, EMU_ORDER);
  while (old < v && !__atomic_compare_exchange_n(p, &old, v, false, EMU_ORDER, EMU_ORDER)) {}
  return old;
}
template <typename T>
T atomicMin(T* p, std::common_type_t<T> v) {
  T old = __atomic_load_n(p, EMU_ORDER);
  while (v < old && !__atomic_compare_exchange_n(p, &old, v, false, EMU_ORDER, EMU_ORDER)) {}
  return old;
}
using std::max;
using std::min;
