// Device helpers shared by the round kernels: the priority key and the
// 64-lane wavefront primitives of CDNA4 (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gcol {

constexpr int kWave = 64;
constexpr int kBlock = 256;          // workgroup of the round kernels: 4 wavefronts
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kAccSlots = 8;         // copies of the launch statistics, kAccStride 64-bit words apart
constexpr int kAccStride = 16;

// Problem kinds (the coloring variants of Section 2.1).
enum Mode : int { kD1 = 1, kD2 = 2, kPD2 = 3 };

// MurmurHash3 32-bit finalizer.  With h = seed-derived constant, the
// priority p(v) = fmix32(gid ^ h) stands for rand(GID) of Algorithm 4: a
// bijection of uint32, so two vertices never draw the same number.
__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

inline uint32_t host_fmix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

inline uint32_t hash_seed(uint32_t seed) { return host_fmix32(seed ^ 0x9E3779B9u); }

// Device-scope (sc1) accesses, performed beyond the XCDs' L2s.  Needed for
// what one workgroup writes and another reads inside one launch: the tail, core
// and batched kernels' hand-overs, counters and flags.  Across launches of a
// stream plain loads see what earlier launches wrote (ld_mut, below), and the
// setup kernels' device-scope accesses there are not needed for that.
template <typename X>
__device__ __forceinline__ X ld_dev(const X* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename X>
__device__ __forceinline__ void st_dev(X* p, X v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Loads of a round kernel's bulk arrays (worklists, lists, offsets, colors,
// bitsets).  The per-round kernels of both engines read them with plain, L2-cacheable loads
// (MUT = 0): the data was written by earlier launches, whose writes every
// later launch on the stream sees (measured on MI355X: 3.8e9 reads of lines
// that another XCD rewrote in the previous launch, none stale), or it is
// written concurrently in ways whose late visibility cannot change a
// result (a compaction that keeps a neighbour committed in the same round, a
// bitset pre-read that only skips an atomic).  Kernels whose phases hand
// data to each other inside one launch (the tail kernel across its grid
// barriers, the persistent batched kernel) read them at device scope
// (MUT = 1).
template <int MUT, typename X>
__device__ __forceinline__ X ld_mut(const X* p) {
  if constexpr (MUT != 0) return ld_dev(p);
  else return *p;
}
template <int MUT, typename X>
__device__ __forceinline__ void st_mut(X* p, X v) {
  if constexpr (MUT != 0) st_dev(p, v);
  else *p = v;
}

// The row of CSR entry e (0 <= e < rp[n]): the last row whose start is <= e,
// by binary search over the n row offsets (empty rows are skipped).
__device__ __forceinline__ int32_t row_of(const int32_t* rp, int32_t n, int32_t e) {
  int32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (rp[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Where a vertex's key comes from.  key(v) = (p(v), gid(v)) packed into 64
// bits so that one unsigned compare is the lexicographic compare; the lower
// key loses a conflict.  With recolorDegrees (Section 3.3) the key is
// (deg(v), p(v), gid(v)); the library then passes each vertex's rank in that
// order, which compares the same way and never ties.
struct KeySource {
  const uint32_t* prio;  // nullable: explicit p(v)
  const int32_t* gid;    // nullable: gid(v) = v
  uint32_t hs;           // hash_seed(seed)
  const uint32_t* rank;  // nullable: recolorDegrees rank (written by an earlier kernel of the call)
};

__device__ __forceinline__ uint64_t key_of(const KeySource& k, int32_t v) {
  if (k.rank) return k.rank[v];
  const uint32_t g = k.gid ? static_cast<uint32_t>(k.gid[v]) : static_cast<uint32_t>(v);
  const uint32_t p = k.prio ? k.prio[v] : fmix32(g ^ k.hs);
  return (static_cast<uint64_t>(p) << 32) | g;
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Workgroups are dispatched round-robin over the 8 XCDs; this renumbering
// gives every XCD a contiguous range of logical ids (grids that are a
// multiple of 8), so each XCD's L2 sees a contiguous range of the work.
__device__ __forceinline__ int32_t xcd_logical_block_of(int32_t nb, int32_t i) {
  const int32_t per = nb / 8;
  if (per == 0 || (nb & 7) != 0) return i;
  return (i & 7) * per + (i >> 3);
}

// Number of set bits of `mask` in lanes below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// x of another lane of its row of 16, by a DPP control word (no LDS access).
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t x) {
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), CTRL, 0xf, 0xf, true));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x >> 32), CTRL, 0xf, 0xf, true));
  return static_cast<uint64_t>(hi) << 32 | lo;
}

// OR of a 64-bit value over aligned groups of G lanes (all lanes of a group
// must be active).  Within a row of 16 lanes by DPP: neighbours, pairs, then
// the mirrored half row and row (whose lanes hold equal values by then).
template <int G>
__device__ __forceinline__ uint64_t group_or(uint64_t x) {
  if constexpr (G >= 2) x |= dpp_u64<0xB1>(x);    // quad_perm 1,0,3,2
  if constexpr (G >= 4) x |= dpp_u64<0x4E>(x);    // quad_perm 2,3,0,1
  if constexpr (G >= 8) x |= dpp_u64<0x141>(x);   // row_half_mirror
  if constexpr (G >= 16) x |= dpp_u64<0x140>(x);  // row_mirror
  if constexpr (G >= 32) x |= __shfl_xor(x, 16, kWave);
  if constexpr (G >= 64) x |= __shfl_xor(x, 32, kWave);
  return x;
}

// 1 if any lane of the calling lane's aligned G-lane group has pred set.
template <int G>
__device__ __forceinline__ bool group_any(bool pred) {
  const uint64_t b = __ballot(pred);
  if (G == kWave) return b != 0;
  const int first = lane_id() & ~(G - 1);
  const uint64_t gm = (G == 64) ? ~0ull : ((1ull << G) - 1ull);
  return ((b >> first) & gm) != 0;
}

__device__ __forceinline__ uint64_t atomic_load_u64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t atomic_load_u32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t atomic_load_i32(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Resets of words that other workgroups update with atomics in the same
// kernel use an atomic read-modify-write too, so that every access to such a
// word (and to its cache line) is performed at the same coherence point;
// a plain store there could leave a dirty partial line in one XCD's L2.
__device__ __forceinline__ void atomic_reset_u32(uint32_t* p) { (void)atomicExch(p, 0u); }
__device__ __forceinline__ void atomic_reset_i32(int32_t* p) { (void)atomicExch(p, 0); }

// The statistics slot of this workgroup (kAccSlots of them, kAccStride apart).
__device__ __forceinline__ unsigned long long* acc_slot(unsigned long long* acc) {
  return acc + kAccStride * (blockIdx.x % kAccSlots);
}

// Orders a wavefront's accesses to LDS before this point and after it, where
// lanes take over words from each other.
__device__ __forceinline__ void wave_step() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Waits until the caller's accesses to memory have completed.  Mutable state
// that only device-scope accesses (performed beyond the L2s) touch is handed
// over by this and a flag; __threadfence also writes the L2 back and
// invalidates it.
__device__ __forceinline__ void wait_own_accesses() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
}

// The first hops of the vertices list[0 .. n) cut into units of at most slice
// entries, dealt to the grid's workgroups in turn: body(i, v, a, z, slices)
// runs for unit [a, z) of v = list[i], which has slices units, with all T
// threads.  T vertices at a time are looked up by the T threads at once; a
// lookup per unit, or a work counter, costs a chain of accesses each.
template <int T>
struct HeavyUnits {
  int32_t wave_sum[T / kWave];
  int32_t end[T];  // units up to and with the vertex
};

template <int T, typename F>
__device__ __forceinline__ void for_heavy_units(const int32_t* rp, const int32_t* list, int32_t n, int32_t slice,
                                                HeavyUnits<T>& sh, F&& body) {
  const int tid = threadIdx.x, wave = tid / kWave;
  int64_t done = 0;  // units of the vertices before i0
  for (int32_t i0 = 0; i0 < n; i0 += T) {
    int32_t incl = 0;
    if (i0 + tid < n) {
      const int32_t v = list[i0 + tid];
      incl = (max(1, rp[v + 1] - rp[v]) - 1) / slice + 1;
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int32_t y = __shfl_up(incl, off, kWave);
      if (lane_id() >= off) incl += y;
    }
    if (lane_id() == kWave - 1) sh.wave_sum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += sh.wave_sum[w];
    sh.end[tid] = incl;
    __syncthreads();
    const int32_t all = sh.end[T - 1];
    int64_t u = (done + gridDim.x - 1 - blockIdx.x) / gridDim.x * gridDim.x + blockIdx.x - done;
    for (; u < all; u += gridDim.x) {
      int r = 0;
#pragma unroll
      for (int step = T / 2; step > 0; step >>= 1) r += sh.end[r + step - 1] <= u ? step : 0;
      const int32_t before = r > 0 ? sh.end[r - 1] : 0;
      const int32_t slices = sh.end[r] - before, j = static_cast<int32_t>(u) - before;
      const int32_t v = list[i0 + r];
      const int32_t q0 = rp[v], q1 = rp[v + 1];
      const int32_t a = q0 + j * slice;
      body(i0 + r, v, a, q1 - a < slice ? q1 : a + slice, slices);
      __syncthreads();
    }
    done += all;
    __syncthreads();
  }
}

}  // namespace gcol
