// Per-vertex steps of one round, shared by the per-graph round kernels and
// the batched persistent kernel: the neighbourhood walk, the first-fit color
// step for a group of G lanes or a whole workgroup, and the detect + commit +
// compact step (Section 3.2, Algorithms 2-4; Section 2.1 and Algorithm 5
// for the distance-2 and partial distance-2 neighbourhoods).
#pragma once

#include <climits>

#include "rounds.hpp"

namespace gcol {

// Loads of the graph arrays.  LD = 0: plain loads (arrays written before the
// call and never rewritten during it).  LD = 1: device-scope loads, for
// graphs whose memory is rewritten by copies between launches of the same
// library instance (the served form's arena), where an XCD's L2 could still
// hold lines of the previous contents.
// MUT (ld_mut): the arrays the rounds write (worklists, colors, work).  0 in
// the per-graph round kernels, whose reads are of earlier launches' writes;
// 1 in the persistent kernel, whose phases hand data over inside one launch.
template <int LD, typename X>
__device__ __forceinline__ X gld(const X* p) {
  if constexpr (LD != 0) return ld_dev(p);
  else return *p;
}

// Visits the neighbourhood entries of v reachable from hop-1 positions
// [beg, end) with lane stride (sub, stride).  get(u) loads what the step needs
// of entry u (0: nothing), use(x) takes it and returns true to stop (checked
// once per batch).  The loops count the entries left: a position behind the
// row's end may not fit 32 bits.  A lane has eight entries in flight, D2/PD2 four of each of
// two second-hop rows: a step's time is its chain of dependent loads (entry,
// then color), so the chain is walked once per eight entries.  Measured on
// MI355X against one entry at a time, with the lanes unchanged: D1 27-point
// 128^3 5.88 -> 3.89 ms, ER n = 10^6 mean degree 16 2.36 -> 1.59 ms, D2
// 7-point 96^3 3.21 -> 1.98 ms.
template <int MODE, int LD = 0, typename GET, typename USE>
__device__ __forceinline__ void scan_nbhd(const GraphView& g, int32_t v, int32_t beg, int32_t end,
                                          int sub, int stride, GET&& get, USE&& use) {
  if constexpr (MODE == kD1) {
    constexpr int N = 8;
    int32_t e0 = beg + sub;
    for (int32_t left = end - beg - sub; left > 0; left -= N * stride, e0 += N * stride) {
      int32_t u[N], x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) u[j] = j * stride < left ? gld<LD>(&g.ci[e0 + j * stride]) : INT_MAX;
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = u[j] < g.limit ? get(u[j]) : 0;
      bool stop = false;
#pragma unroll
      for (int j = 0; j < N; ++j) stop = use(x[j]) || stop;
      if (stop) return;
    }
  } else {
    constexpr int N = 4;
    int32_t e0 = beg + sub;
    for (int32_t left = end - beg - sub; left > 0; left -= 2 * stride, e0 += 2 * stride) {
      int32_t u[2], q[2], n[2], x[2] = {0, 0};
#pragma unroll
      for (int h = 0; h < 2; ++h) u[h] = h * stride < left ? gld<LD>(&g.ci[e0 + h * stride]) : -1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        q[h] = u[h] >= 0 ? gld<LD>(&g.rp2[u[h]]) : 0;
        n[h] = u[h] >= 0 ? gld<LD>(&g.rp2[u[h] + 1]) - q[h] : 0;
        if (MODE == kD2) x[h] = u[h] >= 0 ? get(u[h]) : 0;
      }
      bool stop = false;
      if (MODE == kD2) stop = use(x[0]) || stop, stop = use(x[1]) || stop;
      while (!stop && (n[0] > 0 || n[1] > 0)) {
        int32_t w[2 * N], y[2 * N];
#pragma unroll
        for (int j = 0; j < 2 * N; ++j) w[j] = j % N < n[j / N] ? gld<LD>(&g.ci2[q[j / N] + j % N]) : v;
#pragma unroll
        for (int j = 0; j < 2 * N; ++j) y[j] = w[j] != v ? get(w[j]) : 0;
#pragma unroll
        for (int j = 0; j < 2 * N; ++j) stop = use(y[j]) || stop;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          q[h] += N;
          n[h] -= N;
        }
      }
      if (stop) return;
    }
  }
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

__device__ __forceinline__ int32_t wave_max_i32(int32_t x) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) x = max(x, __shfl_xor(x, off, kWave));
  return x;
}

// ---------------------------------------------------------------------------
// color: group of G lanes per vertex, one chunk of kBlock worklist entries
// ---------------------------------------------------------------------------
template <int MODE, int G, int LD = 0, int MUT = 0>
__device__ __forceinline__ void color_chunk_group(const GraphView& g, const RoundBufs& b, const int32_t* wl, int32_t count,
                                  uint64_t& work_acc) {
  constexpr int per_pass = kBlock / G;
  const int sub = threadIdx.x % G;
  const int32_t* __restrict__ C = b.C;
  int32_t idx = threadIdx.x / G;
  if (idx >= count) return;  // whole groups stay together
  int32_t v = ld_mut<MUT>(&wl[idx]);
  int32_t beg = gld<LD>(&g.rp[v]), end = gld<LD>(&g.rp[v + 1]);
  while (true) {
    // the next vertex's fields are loaded behind this one's scan
    const int32_t next = idx + per_pass;
    const int32_t vn = next < count ? ld_mut<MUT>(&wl[next]) : v;
    int32_t base = 1;
    uint64_t m;
    while (true) {
      m = 0;
      scan_nbhd<MODE, LD>(g, v, beg, end, sub, G, [&](int32_t u) __attribute__((always_inline)) { return ld_mut<MUT>(&C[u]); },
                          [&](int32_t c) __attribute__((always_inline)) {
                            const uint32_t d = static_cast<uint32_t>(c - base);
                            if (d < 64u) m |= 1ull << d;
                            return false;
                          });
      m = group_or<G>(m);
      if (m != ~0ull) break;
      base += 64;
    }
    if (sub == 0) {
      st_dev(&b.T[v], base + static_cast<int32_t>(__builtin_ctzll(~m)));
      work_acc += static_cast<uint64_t>(MODE == kD1 ? end - beg : ld_mut<MUT>(&b.work[v]));
    }
    if (next >= count) break;
    idx = next;
    v = vn;
    beg = gld<LD>(&g.rp[v]);
    end = gld<LD>(&g.rp[v + 1]);
  }
}

// ---------------------------------------------------------------------------
// color: one workgroup per vertex
// ---------------------------------------------------------------------------
template <int MODE, int LD = 0, int MUT = 0>
__device__ __forceinline__ void color_vertex_block(const GraphView& g, const RoundBufs& b, int32_t v,
                                   uint32_t* ovf, uint64_t* red, int32_t* s_min) {
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int32_t beg = gld<LD>(&g.rp[v]), end = gld<LD>(&g.rp[v + 1]);
  const int32_t* __restrict__ C = b.C;
  int32_t base = 1;
  while (true) {
    for (int w = tid; w < kOvfWords; w += kBlock) ovf[w] = 0u;
    if (tid == 0) *s_min = INT_MAX;
    __syncthreads();
    uint64_t m = 0;
    scan_nbhd<MODE, LD>(g, v, beg, end, tid, kBlock, [&](int32_t u) __attribute__((always_inline)) { return ld_mut<MUT>(&C[u]); }, [&](int32_t c) __attribute__((always_inline)) {
      uint32_t d = static_cast<uint32_t>(c - base);
      if (d < 64u) {
        m |= 1ull << d;
      } else {
        d -= 64u;
        if (d < static_cast<uint32_t>(kOvfWords * 32)) atomicOr(&ovf[d >> 5], 1u << (d & 31u));
      }
      return false;
    });
    m = group_or<kWave>(m);
    if (lane_id() == 0) red[wave] = m;
    __syncthreads();
    m = red[0] | red[1] | red[2] | red[3];
    int32_t mex = -1;
    if (m != ~0ull) {
      mex = base + __builtin_ctzll(~m);
    } else {
      for (int w = tid; w < kOvfWords; w += kBlock) {
        const uint32_t x = ovf[w];
        if (x != ~0u) {
          atomicMin(s_min, w * 32 + __builtin_ctz(~x));
          break;
        }
      }
      __syncthreads();
      if (*s_min != INT_MAX) mex = base + 64 + *s_min;
    }
    __syncthreads();
    if (mex > 0) {
      if (tid == 0) st_dev(&b.T[v], mex);
      return;
    }
    base += 64 + kOvfWords * 32;
  }
}

// ---------------------------------------------------------------------------
// detect + commit + compact: group of G lanes per vertex, one chunk
// ---------------------------------------------------------------------------
// Losers of the chunk are collected in LDS (workgroup prefix over the
// wavefront ballots) and given to `out`: out.reserve(n), by one thread, is the
// position of the first, out.put(pos, v) stores one.

// Straight to the next worklist, with one device atomic per chunk.
struct DirectOut {
  int32_t* cnt;
  int32_t* wl;
  __device__ __forceinline__ int32_t reserve(int32_t n) const { return atomicAdd(cnt, n); }
  __device__ __forceinline__ void put(int32_t pos, int32_t v) const { st_dev(&wl[pos], v); }
};

// UNI: every tentative color is 1 and none is read (launch_first_round).
template <int MODE, int G, int LD = 0, int MUT = 0, bool UNI = false, typename Out>
__device__ __forceinline__ void detect_chunk_group(const GraphView& g, const KeySource& k, const RoundBufs& b,
                                   const int32_t* wl, int32_t count, const Out& out, int32_t* s_ent,
                                   int32_t* s_wc, int32_t& maxc_acc) {
  constexpr int per_pass = kBlock / G;
  const int sub = threadIdx.x % G;
  const int32_t* __restrict__ T = b.T;
  int32_t idx = threadIdx.x / G;
  if (idx < count) {
    int32_t v = ld_mut<MUT>(&wl[idx]);
    int32_t beg = gld<LD>(&g.rp[v]), end = gld<LD>(&g.rp[v + 1]), tv = UNI ? 1 : ld_mut<MUT>(&T[v]);
    while (true) {
      const int32_t next = idx + per_pass;
      const int32_t vn = next < count ? ld_mut<MUT>(&wl[next]) : v;
      const uint64_t kv = key_of(k, v);
      bool lose = false;
      // keys first: only higher keys can win
      scan_nbhd<MODE, LD>(g, v, beg, end, sub, G,
                          [&](int32_t u) __attribute__((always_inline)) {
                            if (UNI) return u < g.n && key_of(k, u) > kv ? 1 : 0;
                            return key_of(k, u) > kv ? ld_mut<MUT>(&T[u]) : 0;
                          },
                          [&](int32_t c) __attribute__((always_inline)) {
                            lose = lose || c == tv;
                            return lose;
                          });
      lose = group_any<G>(lose);
      if (sub == 0) {
        if (lose) {
          s_ent[idx] = v;
        } else {
          s_ent[idx] = -1;
          st_dev(&b.C[v], tv);
          maxc_acc = max(maxc_acc, tv);
        }
      }
      if (next >= count) break;
      idx = next;
      v = vn;
      beg = gld<LD>(&g.rp[v]);
      end = gld<LD>(&g.rp[v + 1]);
      tv = UNI ? 1 : ld_mut<MUT>(&T[v]);
    }
  }
  __syncthreads();
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int32_t x = tid < count ? s_ent[tid] : -1;
  const uint64_t bal = __ballot(x >= 0);
  if (lane_id() == 0) s_wc[wave] = static_cast<int32_t>(__popcll(bal));
  __syncthreads();
  if (tid == 0) {
    int32_t tot = 0;
    for (int w = 0; w < kWavesPerBlock; ++w) {
      const int32_t c = s_wc[w];
      s_wc[w] = tot;
      tot += c;
    }
    s_wc[kWavesPerBlock] = tot ? out.reserve(tot) : 0;
  }
  __syncthreads();
  if (x >= 0) out.put(s_wc[kWavesPerBlock] + s_wc[wave] + static_cast<int32_t>(lanes_below(bal)), x);
  __syncthreads();
}

template <int MODE, int LD = 0, int MUT = 0, bool UNI = false>
__device__ __forceinline__ void detect_vertex_block(const GraphView& g, const KeySource& k, const RoundBufs& b,
                                    int32_t v, int32_t off, int32_t& maxc_acc) {
  const int tid = threadIdx.x;
  const int32_t* __restrict__ T = b.T;
  const int32_t tv = UNI ? 1 : ld_mut<MUT>(&T[v]);
  const uint64_t kv = key_of(k, v);
  bool lose = false;
  scan_nbhd<MODE, LD>(g, v, gld<LD>(&g.rp[v]), gld<LD>(&g.rp[v + 1]), tid, kBlock,
                      [&](int32_t u) __attribute__((always_inline)) {
                        if (UNI) return u < g.n && key_of(k, u) > kv ? 1 : 0;
                        return key_of(k, u) > kv ? ld_mut<MUT>(&T[u]) : 0;
                      },
                      [&](int32_t c) __attribute__((always_inline)) {
                        lose = lose || c == tv;
                        return lose;
                      });
  lose = __syncthreads_or(lose);
  if (tid == 0) {
    if (!lose) {
      st_dev(&b.C[v], tv);
      maxc_acc = max(maxc_acc, tv);
    } else {
      const int32_t pos = atomicAdd(&b.cnt_out[kBlockBin], 1);
      st_dev(&b.wl_out[off + pos], v);
    }
  }
}

}  // namespace gcol
