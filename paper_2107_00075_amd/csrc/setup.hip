// Per-call setup kernels: static work and degree bins, initial worklists,
// input-contract validation, the priority hash, and the boundary phase of the
// ghost-layer variant.
#include <algorithm>
#include <climits>

#include "inc.hpp"
#include "setup.hpp"

namespace gcol {

// Sum of 1 + (second-hop row length) over the first-hop entries beg + sub, beg
// + sub + stride, ... below end, eight in flight.  (The entries left are
// counted: a position behind the last may not fit 32 bits.)
__device__ __forceinline__ int64_t hop_work(const GraphView& g, int32_t beg, int32_t end, int32_t sub, int32_t stride) {
  constexpr int N = 8;
  int64_t w = 0;
  int32_t q = beg + sub;
  for (int32_t left = end - beg - sub; left > 0; left -= N * stride, q += N * stride) {
    int32_t u[N], a[N], z[N];
#pragma unroll
    for (int j = 0; j < N; ++j) u[j] = j * stride < left ? g.ci[q + j * stride] : -1;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      a[j] = u[j] >= 0 ? g.rp2[u[j]] : 0;
      z[j] = u[j] >= 0 ? g.rp2[u[j] + 1] : -1;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) w += 1 + (z[j] - a[j]);
  }
  return w;
}

// Adjacency entries one visit of v reads: D1 deg(v); D2 sum over u in N(v)
// of 1 + deg(u); PD2 sum over the rows r of column v of 1 + deg(r) (the
// row entry of the CSC, then the row's columns in the CSR).
template <int MODE>
__device__ __forceinline__ int64_t vertex_work(const GraphView& g, int32_t v) {
  const int32_t b = g.rp[v], e = g.rp[v + 1];
  if (MODE == kD1) return e - b;
  return hop_work(g, b, e, 0, 1);
}

// Bookkeeping of one vertex once its work is known: work, bin, initial colors,
// per-bin counts and the maxima the driver needs.  Called by whole wavefronts
// (wavefront reductions, one atomic per wavefront and quantity).
__device__ void account_vertex(const BinSetup& s, int32_t v, int64_t w, bool active) {
  int bin = -1;
  int32_t c = 0;
  if (active) {
    const int32_t wc = static_cast<int32_t>(w > INT_MAX ? INT_MAX : w);
    st_dev(&s.work[v], wc);
    bin = kBins - 1;
    for (int i = 0; i < kBins - 1; ++i) {
      if (wc <= s.bin_hi[i]) {
        bin = i;
        break;
      }
    }
    st_dev(&s.bin[v], static_cast<int8_t>(bin));
    c = s.init ? ld_dev(&s.init[v]) : 0;
    st_dev(&s.C[v], c);
    st_dev(&s.T[v], c);
  }
  int32_t cmax = c;
  int32_t smax = (active && bin == kSplitBin && c == 0) ? static_cast<int32_t>(w > INT_MAX ? INT_MAX : w) : 0;
  int32_t wmax = (active && c == 0) ? static_cast<int32_t>(w > INT_MAX ? INT_MAX : w) : 0;
  uint64_t wsum = (active && c == 0) ? static_cast<uint64_t>(w) : 0ull;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    cmax = max(cmax, __shfl_xor(cmax, off, kWave));
    smax = max(smax, __shfl_xor(smax, off, kWave));
    wmax = max(wmax, __shfl_xor(wmax, off, kWave));
    wsum += __shfl_xor(wsum, off, kWave);
  }
  if (lane_id() == 0) {
    if (cmax > 0) atomicMax(s.maxc, cmax);
    if (smax > 0) atomicMax(s.max_split_work, smax);
    if (wmax > 0) atomicMax(s.max_work, wmax);
    if (wsum) atomicAdd(s.total_work, static_cast<unsigned long long>(wsum));
  }
  for (int i = 0; i < kBins; ++i) {
    const uint64_t all = __ballot(active && bin == i);
    const uint64_t unc = __ballot(active && bin == i && c == 0);
    if (lane_id() == 0) {
      if (all) atomicAdd(&s.count_all[i], static_cast<int32_t>(__popcll(all)));
      if (unc) atomicAdd(&s.count_unc[i], static_cast<int32_t>(__popcll(unc)));
    }
  }
}

// Per-call totals of the vertices one thread records, flushed once per
// workgroup (a handful of device atomics per workgroup instead of per
// wavefront).
struct BinAcc {
  int32_t cmax = 0, smax = 0, wmax = 0;
  uint64_t wsum = 0;
  int32_t all[kBins] = {0, 0, 0, 0, 0};
  int32_t unc[kBins] = {0, 0, 0, 0, 0};
};

__device__ __forceinline__ void record_vertex(const BinSetup& s, int32_t v, int64_t w, BinAcc& a) {
  const int32_t wc = static_cast<int32_t>(w > INT_MAX ? INT_MAX : w);
  st_dev(&s.work[v], wc);
  int bin = kBins - 1;
  for (int i = 0; i < kBins - 1; ++i) {
    if (wc <= s.bin_hi[i]) {
      bin = i;
      break;
    }
  }
  st_dev(&s.bin[v], static_cast<int8_t>(bin));
  const int32_t c = s.init ? ld_dev(&s.init[v]) : 0;
  st_dev(&s.C[v], c);
  st_dev(&s.T[v], c);
  a.cmax = max(a.cmax, c);
  if (c == 0) {
    if (bin == kSplitBin) a.smax = max(a.smax, wc);
    a.wmax = max(a.wmax, wc);
    a.wsum += static_cast<uint64_t>(w);
  }
#pragma unroll
  for (int i = 0; i < kBins; ++i) {
    a.all[i] += bin == i ? 1 : 0;
    a.unc[i] += (bin == i && c == 0) ? 1 : 0;
  }
}

__device__ void flush_acc(const BinSetup& s, BinAcc& a) {
  __shared__ int32_t s_i[3 + 2 * kBins];
  __shared__ unsigned long long s_sum;
  const int tid = threadIdx.x;
  if (tid < 3 + 2 * kBins) s_i[tid] = 0;
  if (tid == 0) s_sum = 0ull;
  __syncthreads();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    a.cmax = max(a.cmax, __shfl_xor(a.cmax, off, kWave));
    a.smax = max(a.smax, __shfl_xor(a.smax, off, kWave));
    a.wmax = max(a.wmax, __shfl_xor(a.wmax, off, kWave));
    a.wsum += __shfl_xor(a.wsum, off, kWave);
#pragma unroll
    for (int i = 0; i < kBins; ++i) {
      a.all[i] += __shfl_xor(a.all[i], off, kWave);
      a.unc[i] += __shfl_xor(a.unc[i], off, kWave);
    }
  }
  if (lane_id() == 0) {
    atomicMax(&s_i[0], a.cmax);
    atomicMax(&s_i[1], a.smax);
    atomicMax(&s_i[2], a.wmax);
    for (int i = 0; i < kBins; ++i) {
      atomicAdd(&s_i[3 + i], a.all[i]);
      atomicAdd(&s_i[3 + kBins + i], a.unc[i]);
    }
    if (a.wsum) atomicAdd(&s_sum, static_cast<unsigned long long>(a.wsum));
  }
  __syncthreads();
  if (tid == 0) {
    if (s_i[0] > 0) atomicMax(s.maxc, s_i[0]);
    if (s_i[1] > 0) atomicMax(s.max_split_work, s_i[1]);
    if (s_i[2] > 0) atomicMax(s.max_work, s_i[2]);
    if (s_sum) atomicAdd(s.total_work, s_sum);
  } else if (tid <= kBins) {
    const int i = tid - 1;
    if (s_i[3 + i]) atomicAdd(&s.count_all[i], s_i[3 + i]);
    if (s_i[3 + kBins + i]) atomicAdd(&s.count_unc[i], s_i[3 + kBins + i]);
  }
}

constexpr int32_t kThreadHop = 16;  // first-hop entries a thread sums by itself

// A grid-stride loop, one thread per vertex.  D2/PD2 vertices whose first
// hop is longer than kSetupHeavy entries are deferred to heavy_work_kernel.
template <int MODE>
__global__ __launch_bounds__(kBlock) void bin_kernel(GraphView g, BinSetup s) {
  BinAcc acc;
  const int32_t stride = gridDim.x * kBlock;
  for (int32_t base = blockIdx.x * kBlock; base < g.n; base += stride) {
    const int32_t v = base + threadIdx.x;
    bool active = v < g.n;
    bool defer = false;
    if (MODE != kD1 && active) defer = g.rp[v + 1] - g.rp[v] > kSetupHeavy;
    const uint64_t dbal = __ballot(defer);
    if (dbal) {
      const int first = __builtin_ctzll(dbal);
      int32_t b0 = 0;
      if (lane_id() == first) b0 = atomicAdd(s.deferred_cnt, static_cast<int32_t>(__popcll(dbal)));
      b0 = __shfl(b0, first, kWave);
      if (defer) {
        const int32_t di = b0 + static_cast<int32_t>(lanes_below(dbal));
        st_dev(&s.deferred[di], v);
        st_dev(&s.deferred_work[di], 0ull);
        st_dev(&s.deferred_done[di], 0);
      }
    }
    active = active && !defer;
    if (MODE == kD1) {
      if (active) record_vertex(s, v, vertex_work<MODE>(g, v), acc);
    } else {
      // a longer first hop is summed by the whole wavefront (a thread alone
      // walked up to kSetupHeavy entries: 1.06 ms on the 4M x 1M pattern)
      const int32_t q0 = active ? g.rp[v] : 0, q1 = active ? g.rp[v + 1] : 0;
      const bool wide = q1 - q0 > kThreadHop;
      int64_t w = wide ? 0 : hop_work(g, q0, q1, 0, 1);
      uint64_t bal = __ballot(wide);
      while (bal) {
        const int l = __builtin_ctzll(bal);
        bal &= bal - 1ull;
        const int32_t a = __builtin_amdgcn_readlane(q0, l), z = __builtin_amdgcn_readlane(q1, l);
        int64_t x = hop_work(g, a, z, lane_id(), kWave);
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) x += __shfl_xor(x, off, kWave);
        if (lane_id() == l) w = x;
      }
      if (active) record_vertex(s, v, w, acc);
    }
  }
  flush_acc(s, acc);
}

// Deferred heavy vertices: units of up to kHeavySlice first-hop entries; a
// vertex of one unit is recorded at once, the units of a longer one add their
// sums up and the workgroup that completes the last records it.  The sums and
// counters are device-scope, so the hand-over waits for the unit's own
// accesses only.  (With sixteen equal ranges a vertex off one work counter and
// a cache writeback and invalidation per range, the 2236 heavy columns of the
// 4M x 1M PD2 pattern took 2.4 ms.)
constexpr int32_t kHeavySlice = 4096;

template <int MODE>
__global__ __launch_bounds__(kBlock) void heavy_work_kernel(GraphView g, BinSetup s) {
  __shared__ HeavyUnits<kBlock> s_units;
  __shared__ unsigned long long s_sum;
  __shared__ int32_t s_last;
  for_heavy_units<kBlock>(g.rp, s.deferred, ld_dev(s.deferred_cnt), kHeavySlice, s_units,
                          [&](int32_t i, int32_t v, int32_t a, int32_t z, int32_t slices)
                              __attribute__((always_inline)) {
    if (threadIdx.x == 0) s_sum = 0ull;
    __syncthreads();
    uint64_t w = static_cast<uint64_t>(hop_work(g, a, z, static_cast<int32_t>(threadIdx.x), kBlock));
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) w += __shfl_xor(w, off, kWave);
    if (lane_id() == 0 && w) atomicAdd(&s_sum, static_cast<unsigned long long>(w));
    __syncthreads();
    if (threadIdx.x == 0) {
      s_last = 1;
      if (slices > 1) {
        atomicAdd(&s.deferred_work[i], s_sum);
        wait_own_accesses();
        s_last = atomicAdd(&s.deferred_done[i], 1) == slices - 1 ? 1 : 0;
        if (s_last) s_sum = ld_dev(&s.deferred_work[i]);
      }
    }
    __syncthreads();
    if (s_last && threadIdx.x < kWave) account_vertex(s, v, static_cast<int64_t>(s_sum), threadIdx.x == 0);
  });
}

// Appends every uncolored vertex (C[v] == 0) to its bin's region of the
// worklist; split vertices get a split index (their position in the split
// region) and the region holds indices.  Each workgroup owns a contiguous
// range of per_block vertices: it counts its vertices per bin, reserves its
// slots with one device atomic per bin, then writes them.
__global__ __launch_bounds__(kBlock) void scatter_kernel(int32_t n, const int32_t* C, const int8_t* binv,
                                                         BinLayout L, int32_t* wl, int32_t* cnt,
                                                         int32_t* split_vertex, int32_t per_block) {
  __shared__ int32_t s_cnt[kBins][kWavesPerBlock];
  __shared__ int32_t s_next[kBins];
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int32_t lo = blockIdx.x * per_block;
  const int32_t hi = min(n, lo + per_block);
  int32_t my[kBins] = {0, 0, 0, 0, 0};
  for (int32_t v = lo + tid; v < hi; v += kBlock) {
    const bool active = ld_mut<0>(&C[v]) == 0;
    const int bin = active ? static_cast<int>(ld_mut<0>(&binv[v])) : -1;
#pragma unroll
    for (int i = 0; i < kBins; ++i) my[i] += bin == i ? 1 : 0;
  }
#pragma unroll
  for (int i = 0; i < kBins; ++i) {
    int32_t x = my[i];
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) x += __shfl_xor(x, off, kWave);
    if (lane_id() == 0) s_cnt[i][wave] = x;
  }
  __syncthreads();
  if (tid < kBins) {
    int32_t tot = 0;
    for (int w = 0; w < kWavesPerBlock; ++w) tot += s_cnt[tid][w];
    s_next[tid] = tot ? atomicAdd(&cnt[tid], tot) : 0;
  }
  __syncthreads();
  for (int32_t base = lo; base < hi; base += kBlock) {
    const int32_t v = base + tid;
    const bool active = v < hi && ld_mut<0>(&C[v]) == 0;
    const int bin = active ? static_cast<int>(ld_mut<0>(&binv[v])) : -1;
    int32_t rank = 0;
#pragma unroll
    for (int i = 0; i < kBins; ++i) {
      const uint64_t bal = __ballot(bin == i);
      if (bin == i) rank = static_cast<int32_t>(lanes_below(bal));
      if (lane_id() == 0) s_cnt[i][wave] = static_cast<int32_t>(__popcll(bal));
    }
    __syncthreads();
    if (active) {
      int32_t pos = s_next[bin] + rank;
      for (int w = 0; w < wave; ++w) pos += s_cnt[bin][w];
      if (bin == kSplitBin) {
        st_dev(&split_vertex[pos], v);
        st_dev(&wl[L.off[bin] + pos], pos);
      } else {
        st_dev(&wl[L.off[bin] + pos], v);
      }
    }
    __syncthreads();
    if (tid < kBins) {
      int32_t tot = 0;
      for (int w = 0; w < kWavesPerBlock; ++w) tot += s_cnt[tid][w];
      s_next[tid] += tot;
    }
    __syncthreads();
  }
}

__device__ void validate_row(int32_t v, int32_t n_cols, const int32_t* rp, const int32_t* ci,
                             const int32_t* rpT, const int32_t* ciT, int32_t n_trows, int square,
                             int32_t* err);

// Input contract (COLOR_FLAG_VALIDATE).  Rows strictly increasing, ids in
// range, no self-loops when `square`, and every entry (v, u) mirrored as
// (u, v) in the transpose arrays (rpT, ciT) — for D1/D2 the adjacency itself,
// for PD2 the CSC of the same pattern.
__global__ __launch_bounds__(kBlock) void validate_kernel(int32_t n_rows, int32_t n_cols, const int32_t* rp,
                                                          const int32_t* ci, const int32_t* rpT,
                                                          const int32_t* ciT, int32_t n_trows, int square,
                                                          int32_t* err) {
  const int32_t v = blockIdx.x * kBlock + threadIdx.x;
  if (v < n_rows) validate_row(v, n_cols, rp, ci, rpT, ciT, n_trows, square, err);
}

__device__ void validate_row(int32_t v, int32_t n_cols, const int32_t* rp, const int32_t* ci,
                             const int32_t* rpT, const int32_t* ciT, int32_t n_trows, int square,
                             int32_t* err) {
  const int32_t b = rp[v], e = rp[v + 1];
  if (b > e) {
    atomicOr(err, 1);
    return;
  }
  int32_t prev = -1;
  for (int32_t q = b; q < e; ++q) {
    const int32_t u = ci[q];
    if (u < 0 || u >= n_cols) {
      atomicOr(err, 2);
      return;
    }
    if (u <= prev) atomicOr(err, 4);
    if (square && u == v) atomicOr(err, 8);
    prev = u;
    if (u >= n_trows) continue;  // no transpose row for u (e.g. a ghost without a row)
    // binary search v in the transpose row of u
    int32_t lo = rpT[u], hi = rpT[u + 1] - 1;
    bool found = false;
    while (lo <= hi) {
      const int32_t mid = lo + ((hi - lo) >> 1);
      const int32_t x = ciT[mid];
      if (x == v) {
        found = true;
        break;
      }
      if (x < v) lo = mid + 1;
      else hi = mid - 1;
    }
    if (!found) atomicOr(err, 16);
  }
}

__global__ __launch_bounds__(kBlock) void check_rowptr_kernel(int32_t n, const int32_t* rp, int32_t* err) {
  const int32_t v = blockIdx.x * kBlock + threadIdx.x;
  if (v == 0 && rp[0] != 0) atomicOr(err, 1);
  if (v < n && rp[v] > rp[v + 1]) atomicOr(err, 1);
}

__global__ __launch_bounds__(kBlock) void priority_kernel(int32_t n, const int32_t* gid, uint32_t hs,
                                                          uint32_t* out) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) {
    const uint32_t g = gid ? static_cast<uint32_t>(gid[i]) : static_cast<uint32_t>(i);
    st_dev(&out[i], fmix32(g ^ hs));
  }
}

// Ghost phase 2 (Algorithm 3 with Algorithm 4 on the ghosts' fixed colors):
// every owned-ghost edge with equal colors is a conflict; the owned endpoint
// loses when the ghost's key is greater, otherwise the ghost is flagged.  All
// pairs are judged on the phase-1 colors; losers are uncolored afterwards by
// recolor_begin_kernel.  loser and gflag must be zeroed first.  A workgroup
// takes kBoundaryEntries consecutive owned-row entries, so that a hub's row
// spreads over many, with the offsets of their rows in LDS.  (A binary search
// of all rows in memory per entry took 103 us on a sixteenth of RMAT
// scale 22.)
constexpr int kBoundaryPer = 8;
constexpr int kBoundaryEntries = kBoundaryPer * kBlock;
constexpr int kBoundaryRows = 2048;

__global__ __launch_bounds__(kBlock) void boundary_kernel(int32_t n_owned, const int32_t* rp,
                                                          const int32_t* ci, const int32_t* C,
                                                          const int32_t* ghost_colors, KeySource k,
                                                          int32_t* loser, int32_t* gflag,
                                                          unsigned long long* conflicts) {
  __shared__ int32_t s_rp[kBoundaryRows];
  __shared__ int32_t s_found;
  constexpr int N = kBoundaryPer;
  const int tid = threadIdx.x;
  const int32_t nnz = rp[n_owned];
  const int32_t e0 = blockIdx.x * kBoundaryEntries;
  if (e0 >= nnz) return;
  const int32_t e1 = nnz - e0 < kBoundaryEntries ? nnz : e0 + kBoundaryEntries;
  int32_t u[N], gc[N], v[N], cv[N];
#pragma unroll
  for (int j = 0; j < N; ++j) u[j] = e0 + j * kBlock + tid < e1 ? ci[e0 + j * kBlock + tid] : 0;
  const int32_t lo = row_of(rp, n_owned, e0);
  const int32_t rows = row_of(rp, n_owned, e1 - 1) - lo + 1;
  const bool lds = rows <= kBoundaryRows;  // beyond (mostly empty rows): searched in memory
  if (tid == 0) s_found = 0;
  for (int i = tid; lds && i < rows; i += kBlock) s_rp[i] = rp[lo + i];
#pragma unroll
  for (int j = 0; j < N; ++j) gc[j] = u[j] >= n_owned ? ghost_colors[u[j] - n_owned] : 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < N; ++j)
    v[j] = lds ? row_of(s_rp, rows, e0 + j * kBlock + tid) : row_of(rp + lo, rows, e0 + j * kBlock + tid);
#pragma unroll
  for (int j = 0; j < N; ++j) cv[j] = u[j] >= n_owned ? ld_dev(&C[lo + v[j]]) : 0;
  int32_t found = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if (u[j] < n_owned || gc[j] != cv[j]) continue;
    ++found;
    if (key_of(k, u[j]) > key_of(k, lo + v[j])) st_dev(&loser[lo + v[j]], 1);
    else st_dev(&gflag[u[j] - n_owned], 1);
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) found += __shfl_xor(found, off, kWave);
  if (lane_id() == 0 && found) atomicAdd(&s_found, found);
  __syncthreads();
  if (tid == 0 && s_found) atomicAdd(conflicts, static_cast<unsigned long long>(s_found));
}

// Distance-2 / partial distance-2 ghost phase 2 (Algorithm 5 over the owned
// vertices): every owned vertex's two-hop walk is compared with the ghosts'
// fixed colors, a thread per hop-1 entry (u) walking u itself (D2) and u's
// hop-2 row, so heavy vertices spread over many threads.  A conflicting
// ghost x of v makes v lose (key(x) > key(v)) or flags x; both are
// idempotent, so the walk's repeated entries do not matter to them.  The
// count is of distinct (v, x) pairs: pass 1 counts the conflicting entries,
// pass 2 inserts them into an open-addressing set of (v, x) keys sized for
// them and counts the insertions that found an empty slot.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <int MODE>
__global__ __launch_bounds__(kBlock) void boundary2_kernel(GraphView g, int32_t n_owned, const int32_t* C,
                                                           const int32_t* ghost_colors, KeySource k, int32_t* loser,
                                                           int32_t* gflag, unsigned long long* hits,
                                                           unsigned long long* set, uint64_t set_mask,
                                                           unsigned long long* conflicts) {
  const int32_t e = blockIdx.x * kBlock + threadIdx.x;
  const int32_t nnz1 = g.rp[n_owned];
  uint64_t n_hit = 0, n_new = 0;
  if (e < nnz1) {
    const int32_t v = row_of(g.rp, n_owned, e);
    const int32_t cv = ld_dev(&C[v]);
    const int32_t u = g.ci[e];
    auto visit = [&](int32_t x) {
      if (x < n_owned || x == v || ghost_colors[x - n_owned] != cv) return;
      ++n_hit;
      if (key_of(k, x) > key_of(k, v)) st_dev(&loser[v], 1);
      else st_dev(&gflag[x - n_owned], 1);
      if (set) {
        const unsigned long long pair = (static_cast<unsigned long long>(v) << 32) | static_cast<uint32_t>(x);
        for (uint64_t h = mix64(pair) & set_mask;; h = (h + 1) & set_mask) {
          const unsigned long long was = atomicCAS(&set[h], ~0ull, pair);
          if (was == ~0ull) {
            ++n_new;
            break;
          }
          if (was == pair) break;
        }
      }
    };
    if (MODE == kD2) visit(u);
    for (int32_t q = g.rp2[u]; q < g.rp2[u + 1]; ++q) visit(g.ci2[q]);
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    n_hit += __shfl_xor(n_hit, off, kWave);
    n_new += __shfl_xor(n_new, off, kWave);
  }
  if (lane_id() == 0) {
    if (n_hit) atomicAdd(hits, static_cast<unsigned long long>(n_hit));
    if (n_new) atomicAdd(conflicts, static_cast<unsigned long long>(n_new));
  }
}

__global__ __launch_bounds__(kBlock) void fill_u64_kernel(unsigned long long* p, uint64_t n, unsigned long long x) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (i < n) p[i] = x;
}

// Block totals of a grid-stride ghost kernel: one atomic per workgroup (one
// per wavefront on the same word took 159 us for 3.9 million ghosts).
__device__ __forceinline__ void flush_max_count(int32_t mx, uint32_t count, int32_t* max_out,
                                                unsigned long long* count_out) {
  __shared__ int32_t s_max;
  __shared__ uint32_t s_count;
  if (threadIdx.x == 0) {
    s_max = 0;
    s_count = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    mx = max(mx, __shfl_xor(mx, off, kWave));
    count += __shfl_xor(count, off, kWave);
  }
  if (lane_id() == 0) {
    if (mx > 0) atomicMax(&s_max, mx);
    if (count) atomicAdd(&s_count, count);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_max > 0) atomicMax(max_out, s_max);
    if (s_count) atomicAdd(count_out, static_cast<unsigned long long>(s_count));
  }
}

__global__ __launch_bounds__(kBlock) void ghost_begin_kernel(int32_t n_owned, int32_t n_ghost, const int32_t* init,
                                                             int32_t* C, int32_t* T, int32_t* loser, int32_t* gflag,
                                                             int32_t* maxc, unsigned long long* uncolored) {
  int32_t mx = 0;
  uint32_t zeros = 0;
  const int64_t items = max(n_owned, n_ghost), stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < items; i += stride) {
    if (i < n_ghost) st_dev(&gflag[i], 0);
    if (i >= n_owned) continue;
    st_dev(&loser[i], 0);
    if (init) {
      const int32_t c = init[i];
      st_dev(&C[i], c);
      st_dev(&T[i], c);
      mx = max(mx, c);
      zeros += c == 0;
    }
  }
  flush_max_count(mx, zeros, maxc, uncolored);
}

__global__ __launch_bounds__(kBlock) void recolor_begin_kernel(int32_t n_owned, int32_t n_ghost, const int32_t* loser,
                                                               const int32_t* ghost_colors, int32_t* C, int32_t* T,
                                                               int32_t* maxc, uint32_t* zero, int zero_words) {
  int32_t mx = 0;
  const int64_t items = max(max(n_owned, n_ghost), zero_words), stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < items; i += stride) {
    if (i < zero_words) st_dev(&zero[i], 0u);
    if (i < n_owned && ld_dev(&loser[i])) st_dev(&C[i], 0);
    if (i < n_ghost) {
      const int32_t c = ghost_colors[i];
      st_dev(&C[n_owned + i], c);
      st_dev(&T[n_owned + i], c);
      mx = max(mx, c);
    }
  }
  flush_max_count(mx, 0u, maxc, nullptr);
}

__global__ __launch_bounds__(kBlock) void ghost_out_kernel(int32_t n_owned, int32_t n_ghost, const int32_t* C,
                                                           const int32_t* gflag, int32_t* owned_colors,
                                                           uint8_t* remote_loser, int32_t* max_color,
                                                           unsigned long long* remote) {
  int32_t mx = 0;
  uint32_t flags = 0;
  const int64_t items = max(n_owned, n_ghost), stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < items; i += stride) {
    if (i < n_owned) {
      const int32_t c = ld_dev(&C[i]);
      st_dev(&owned_colors[i], c);
      mx = max(mx, c);
    }
    if (i < n_ghost) {
      const bool f = ld_dev(&gflag[i]) != 0;
      if (remote_loser) remote_loser[i] = f ? 1 : 0;
      flags += f;
    }
  }
  flush_max_count(mx, flags, max_color, remote);
}

static inline int blocks_for(int64_t n) { return static_cast<int>((n + kBlock - 1) / kBlock); }

// Grid caps of the setup kernels.  Every workgroup of the bin setup adds its
// totals to the same few words, about 10 ns each: 512 workgroups take 30 us on
// a 2 M-vertex mesh, 2048 39 us; the worklist scatter (one word) is no faster
// with fewer.
constexpr int kSetupGrid = 512;
constexpr int kScatterGrid = 2048;

template <int MODE>
void launch_bin(const GraphView& g, const BinSetup& s, hipStream_t st) {
  if (g.n <= 0) return;
  hipLaunchKernelGGL(bin_kernel<MODE>, dim3(std::min(blocks_for(g.n), kSetupGrid)), dim3(kBlock), 0, st, g, s);
  if (MODE != kD1)
    hipLaunchKernelGGL(heavy_work_kernel<MODE>, dim3(std::min(blocks_for(g.n), 512)), dim3(kBlock), 0, st, g, s);
}
template void launch_bin<kD1>(const GraphView&, const BinSetup&, hipStream_t);
template void launch_bin<kD2>(const GraphView&, const BinSetup&, hipStream_t);
template void launch_bin<kPD2>(const GraphView&, const BinSetup&, hipStream_t);

void launch_scatter(int32_t n, const int32_t* C, const int8_t* bin, const BinLayout& L, int32_t* wl,
                    int32_t* cnt, int32_t* split_vertex, hipStream_t st) {
  if (n <= 0) return;
  const int blocks = std::min(blocks_for(n), kScatterGrid);
  const int64_t per = (static_cast<int64_t>(n) + blocks - 1) / blocks;
  const int32_t per_block = static_cast<int32_t>((per + kBlock - 1) / kBlock * kBlock);
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks), dim3(kBlock), 0, st, n, C, bin, L, wl, cnt, split_vertex,
                     per_block);
}

void launch_validate(int32_t n_rows, int32_t n_cols, const int32_t* rp, const int32_t* ci,
                     const int32_t* rpT, const int32_t* ciT, int32_t n_trows, int square, int32_t* err,
                     hipStream_t st) {
  hipLaunchKernelGGL(check_rowptr_kernel, dim3(blocks_for(static_cast<int64_t>(n_rows) + 1)), dim3(kBlock),
                     0, st, n_rows, rp, err);
  if (n_rows > 0)
    hipLaunchKernelGGL(validate_kernel, dim3(blocks_for(n_rows)), dim3(kBlock), 0, st, n_rows, n_cols, rp,
                       ci, rpT, ciT, n_trows, square, err);
}

void launch_priority(int32_t n, const int32_t* gid, uint32_t hs, uint32_t* out, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(priority_kernel, dim3(blocks_for(n)), dim3(kBlock), 0, st, n, gid, hs, out);
}

void launch_boundary(int32_t n_owned, int32_t owned_nnz, const int32_t* rp, const int32_t* ci, const int32_t* C,
                     const int32_t* ghost_colors, const KeySource& k, int32_t* loser, int32_t* gflag,
                     unsigned long long* conflicts, hipStream_t st) {
  if (n_owned > 0 && owned_nnz > 0)
    hipLaunchKernelGGL(boundary_kernel, dim3((owned_nnz - 1) / kBoundaryEntries + 1), dim3(kBlock), 0, st, n_owned, rp, ci, C,
                       ghost_colors, k, loser, gflag, conflicts);
}

// The grid-stride ghost kernels: a workgroup per 1024 items, up to 1024.
static inline int ghost_grid(int64_t n) { return static_cast<int>(std::min<int64_t>((n + 1023) / 1024, 1024)); }

void launch_ghost_begin(int32_t n_owned, int32_t n_ghost, const int32_t* init, int32_t* C, int32_t* T, int32_t* loser,
                        int32_t* gflag, int32_t* maxc, unsigned long long* uncolored, hipStream_t st) {
  hipLaunchKernelGGL(ghost_begin_kernel, dim3(ghost_grid(std::max(n_owned, n_ghost))), dim3(kBlock), 0, st, n_owned,
                     n_ghost, init, C, T, loser, gflag, maxc, uncolored);
}

void launch_recolor_begin(int32_t n_owned, int32_t n_ghost, const int32_t* loser, const int32_t* gc, int32_t* C,
                          int32_t* T, int32_t* maxc, uint32_t* zero, int zero_words, hipStream_t st) {
  hipLaunchKernelGGL(recolor_begin_kernel, dim3(ghost_grid(std::max(std::max(n_owned, n_ghost), zero_words))),
                     dim3(kBlock), 0, st, n_owned, n_ghost, loser, gc, C, T, maxc, zero, zero_words);
}

void launch_ghost_out(int32_t n_owned, int32_t n_ghost, const int32_t* C, const int32_t* gflag, int32_t* owned_colors,
                      uint8_t* remote_loser, int32_t* max_color, unsigned long long* remote, hipStream_t st) {
  hipLaunchKernelGGL(ghost_out_kernel, dim3(ghost_grid(std::max(n_owned, n_ghost))), dim3(kBlock), 0, st, n_owned,
                     n_ghost, C, gflag, owned_colors, remote_loser, max_color, remote);
}

// Ghost phase 1 reads the owned-induced subgraph: the owned rows without
// their ghost entries (ids >= n_owned).  A flag per owned-row entry (1: kept),
// an exclusive scan of the flags, then every kept entry moves to its scanned
// position and every row starts at the scan of its first entry.
__global__ __launch_bounds__(kBlock) void owned_flags_kernel(int32_t n_owned, const int32_t* rp, const int32_t* ci,
                                                             int32_t* flag) {
  const int32_t e = blockIdx.x * kBlock + threadIdx.x;
  const int32_t nnz = rp[n_owned];
  if (e < nnz) st_dev(&flag[e], ci[e] < n_owned ? 1 : 0);
  else if (e == nnz) st_dev(&flag[e], 0);
}

__global__ __launch_bounds__(kBlock) void owned_compact_kernel(int32_t n_owned, const int32_t* rp, const int32_t* ci,
                                                               const int32_t* pos, int32_t* rp1, int32_t* ci1) {
  const int32_t e = blockIdx.x * kBlock + threadIdx.x;
  if (e <= n_owned) st_dev(&rp1[e], pos[rp[e]]);
  if (e < rp[n_owned] && ci[e] < n_owned) st_dev(&ci1[pos[e]], ci[e]);
}

// Tentative ghost recoloring, one layer: a ghost's row in the local graph is
// the owned vertices adjacent to it (the local graph's undirected
// owned-ghost edges).  Counts them per ghost ...
__global__ __launch_bounds__(kBlock) void ghost_row_count_kernel(int32_t n_owned, const int32_t* rp,
                                                                 const int32_t* ci, int32_t* cnt) {
  const int32_t e = blockIdx.x * kBlock + threadIdx.x;  // a thread per owned-row entry
  if (e >= rp[n_owned]) return;
  const int32_t u = ci[e];
  if (u >= n_owned) atomicAdd(&cnt[u - n_owned], 1);
}

// ... and, with the per-ghost offsets goff (exclusive scan of the counts,
// n_ghost + 1 entries), writes the local CSR over all owned + ghost ids:
// owned rows as given, then the ghosts' rows.
__global__ __launch_bounds__(kBlock) void ghost_rows_kernel(int32_t n_owned, int32_t n_ghost, const int32_t* rp,
                                                            const int32_t* ci, const int32_t* goff, int32_t* fill,
                                                            int32_t* rp3, int32_t* ci3) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;  // offsets by id, entries by position
  const int32_t owned_nnz = rp[n_owned];
  if (i <= n_owned) st_dev(&rp3[i], rp[i]);
  if (i > 0 && i <= n_ghost) st_dev(&rp3[n_owned + i], owned_nnz + goff[i]);
  if (i >= owned_nnz) return;
  const int32_t u = ci[i];
  st_dev(&ci3[i], u);
  if (u >= n_owned) {
    const int32_t j = u - n_owned;
    st_dev(&ci3[owned_nnz + goff[j] + atomicAdd(&fill[j], 1)], row_of(rp, n_owned, i));
  }
}

// Colors the recoloring phase starts from, for the rows-carrying ids
// [0, n3): owned vertices as committed (losers already 0), ghosts as
// received except the losing ones (0: recolored tentatively); a ghost whose
// color is not known yet (0 received) gets kGhostUnknown, which keeps it out
// of the worklist and out of every first fit.
__global__ __launch_bounds__(kBlock) void ghost_recolor_init_kernel(int32_t n_owned, int32_t n3, const int32_t* C,
                                                                    const int32_t* gc, const int32_t* gflag,
                                                                    int32_t* init) {
  const int32_t v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n3) return;
  int32_t c;
  if (v < n_owned) {
    c = ld_dev(&C[v]);
  } else {
    const int32_t j = v - n_owned;
    c = ld_dev(&gflag[j]) ? 0 : (gc[j] == 0 ? kGhostUnknown : gc[j]);
  }
  st_dev(&init[v], c);
}

void launch_ghost_rows(int32_t n_owned, int32_t n_ghost, int32_t owned_nnz, const int32_t* rp, const int32_t* ci,
                       int32_t* cnt, int32_t* goff, int32_t* fill, int32_t* rp3, int32_t* ci3, void* scan_tmp,
                       size_t scan_bytes, hipStream_t st, int* err) {
  *err = 0;
  if (n_ghost > 0) {
    hipLaunchKernelGGL(ghost_row_count_kernel, dim3(blocks_for(std::max(owned_nnz, 1))), dim3(kBlock), 0, st,
                       n_owned, rp, ci, cnt);
    if (exclusive_scan_i32(cnt, goff, n_ghost + 1, scan_tmp, &scan_bytes, st)) *err = 1;
  }
  const int32_t items = std::max(std::max(n_owned + 1, n_ghost + 1), owned_nnz);
  hipLaunchKernelGGL(ghost_rows_kernel, dim3(blocks_for(items)), dim3(kBlock), 0, st, n_owned, n_ghost, rp, ci,
                     goff, fill, rp3, ci3);
}

int launch_owned_subgraph(int32_t n_owned, int32_t owned_nnz, const int32_t* rp, const int32_t* ci, int32_t* flag,
                          int32_t* pos, int32_t* rp1, int32_t* ci1_or_null, void* scan_tmp, size_t scan_bytes,
                          hipStream_t st) {
  const int32_t items = std::max(owned_nnz + 1, n_owned + 1);
  if (ci1_or_null == nullptr) {
    hipLaunchKernelGGL(owned_flags_kernel, dim3(blocks_for(owned_nnz + 1)), dim3(kBlock), 0, st, n_owned, rp, ci, flag);
    return exclusive_scan_i32(flag, pos, owned_nnz + 1, scan_tmp, &scan_bytes, st);
  }
  hipLaunchKernelGGL(owned_compact_kernel, dim3(blocks_for(items)), dim3(kBlock), 0, st, n_owned, rp, ci, pos, rp1,
                     ci1_or_null);
  return 0;
}

void launch_ghost_recolor_init(int32_t n_owned, int32_t n3, const int32_t* C, const int32_t* gc, const int32_t* gflag,
                               int32_t* init, hipStream_t st) {
  if (n3 > 0)
    hipLaunchKernelGGL(ghost_recolor_init_kernel, dim3(blocks_for(n3)), dim3(kBlock), 0, st, n_owned, n3, C, gc,
                       gflag, init);
}

void launch_fill_u64(unsigned long long* p, uint64_t n, unsigned long long x, hipStream_t st) {
  if (n > 0)
    hipLaunchKernelGGL(fill_u64_kernel, dim3(static_cast<unsigned>((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, p,
                       n, x);
}

template <int MODE>
void launch_boundary2(const GraphView& g, int32_t n_owned, int32_t nnz1, const int32_t* C, const int32_t* ghost_colors,
                      const KeySource& k, int32_t* loser, int32_t* gflag, unsigned long long* hits,
                      unsigned long long* set, uint64_t set_mask, unsigned long long* conflicts, hipStream_t st) {
  if (nnz1 > 0)
    hipLaunchKernelGGL(boundary2_kernel<MODE>, dim3(blocks_for(nnz1)), dim3(kBlock), 0, st, g, n_owned, C,
                       ghost_colors, k, loser, gflag, hits, set, set_mask, conflicts);
}
template void launch_boundary2<kD2>(const GraphView&, int32_t, int32_t, const int32_t*, const int32_t*,
                                    const KeySource&, int32_t*, int32_t*, unsigned long long*, unsigned long long*,
                                    uint64_t, unsigned long long*, hipStream_t);
template void launch_boundary2<kPD2>(const GraphView&, int32_t, int32_t, const int32_t*, const int32_t*,
                                     const KeySource&, int32_t*, int32_t*, unsigned long long*, unsigned long long*,
                                     uint64_t, unsigned long long*, hipStream_t);

}  // namespace gcol
