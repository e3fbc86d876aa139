// Core kernels: the remaining synchronous rounds once the worklist fits the
// chip's registers as a bit matrix.
//
// The last rounds of a skewed graph or a dense two-hop graph are many and
// small: the vertices left form a dense core that commits a few vertices per
// round.  There a round's time is latency: the tail kernel's chain of about
// twenty dependent device-scope accesses and two grid barriers takes 40-50 us
// whether the round holds 10^4 vertices or ten.
//
// core_rank_kernel numbers the vertices left by key, highest first, and
// core_build_kernel turns each one's active list into a row of bits over
// those numbers.  core_kernel then runs all rounds on the rows:
//
//  * A workgroup owns 64 or 96 consecutive numbers; a row lives in the
//    registers of one wavefront, its words interleaved over the lanes.  "A
//    neighbour of higher key" is the part of the row below the vertex's own
//    number.
//  * Phase A of a round publishes, per color c in use, the bits of the
//    vertices whose tentative color is c.  A vertex loses iff its row meets
//    the bits of its own color below its own number.
//  * Phase B publishes the bits of the vertices that committed in the round
//    and their colors, packed.  A workgroup reads of each such vertex's row
//    only the words of its own vertices (the rows are symmetric) and adds the
//    color to the forbidden colors of the neighbours it has, a window of 64
//    colors from about the tentative color on.  A loser then moves to the
//    first color from its tentative color on that its window does not hold.
//    That is its first fit in the next round: forbidden colors only grow, so
//    a tentative color never decreases; and a color committed in a round is
//    less than kCoreSlots above every tentative color, inside the window.
//  * Every published 64-bit word carries the round number in its upper half
//    and 32 vertices' bits in its lower half, so a reader polls the data
//    itself: one store and one load per exchange, with no flag, counter or
//    fence.  A word is rewritten only after every workgroup has read it: a
//    workgroup publishes phase A of round r+1 after it has seen every
//    workgroup's phase B summary word of round r, and those are published
//    after the writer has read phase A of round r (and the same with the
//    phases exchanged).
//  * Color c travels in slot c mod kCoreSlots.  The tentative colors in use
//    span few colors (at most 10 on R-MAT, power-law and dense random graphs
//    of every size tried); if they ever span more than the slots, every
//    workgroup sees it in the same round's summary words and the launch ends
//    having written nothing, and the rounds go on in the tail kernel, down to
//    the one-workgroup stage, which takes any spread.
//  * As the worklist shrinks, the rows are compacted to the vertices left
//    (core_stage's hand-over): at 4096 vertices to 64 workgroups with 128-word
//    rows, at 1024 to one workgroup, a thread per vertex, which needs no
//    exchange: its rounds meet at workgroup barriers and take 2-4 us.
//
// Bound: latency of the exchanges, then of LDS.
#include <algorithm>
#include <climits>

#include "core.hpp"
#include "grid_sync.hpp"

namespace gcol {

namespace {

constexpr int kCoreThreads = 1024;
constexpr int kCoreWaves = kCoreThreads / kWave;
constexpr int kRankPer = 128;           // vertices numbered by one workgroup
constexpr int kRankChunk = 4096;        // keys staged in LDS at a time
constexpr int32_t kCoreMaxColor = 1 << 20;  // tentative colors a summary word can carry
constexpr int32_t kMidMax = kCoreMid;   // vertices of the second stage
constexpr int32_t kSmallMax = kCoreSmall;  // vertices of the one-workgroup stage

// Row words (stride of the row array) of a stage over n vertices.
__host__ __device__ constexpr int32_t row_words(int32_t n) {
  return n <= kSmallMax ? kSmallMax / 32 : n <= kMidMax ? kMidMax / 32 : n <= 16384 ? 512 : 768;
}

struct CoreWorklist {
  const int32_t* wl;
  int32_t off[kBins];
  int32_t cnt[kBins];
};

__device__ __forceinline__ int32_t core_entry(const CoreWorklist& q, int32_t i) {
  int bin = 0;
  while (bin < kBins - 1 && i >= q.cnt[bin]) {
    i -= q.cnt[bin];
    ++bin;
  }
  return q.wl[q.off[bin] + i];
}

// A stage's vertices in key order: id, tentative color t, the forbidden
// colors [t, t + 64) as bits, and the row.
struct CoreSet {
  int32_t* v;
  int32_t* t;
  uint64_t* fw;
  uint32_t* rows;
};

// A stage's exchange words: [slot][word] of phase A and [kCoreColorWords][word]
// of phase B (the slots of the committed colors, six to a word), their summary
// words [word] (phase B: the vertices that committed), and a flag per
// workgroup set at the hand-over.
constexpr int kCoreColors = 6;                          // 5-bit slots in a word
constexpr int kCoreColorWords = (32 + kCoreColors - 1) / kCoreColors;

struct CoreExchange {
  uint64_t* A;
  uint64_t* B;
  uint64_t* ma;
  uint64_t* mb;
  uint64_t* flag;
};

constexpr int kSets = 3;  // the first stage's, the second's and the one-workgroup stage's

struct CoreScratch {
  CoreSet set[kSets];
  CoreExchange x[kSets - 1];
};

// Word w of v's forbidden bitset, 0 (all free) beyond its end.
__device__ __forceinline__ uint32_t core_word(const IncBufs& b, int32_t v, int32_t w) {
  if (w == 0) return b.F[v];
  const int32_t w0 = b.fw_off[v];
  return w <= b.fw_off[v + 1] - w0 ? b.Fx[w0 + w - 1] : 0u;
}

// Adds color c to v's forbidden bitset, which only the calling thread reads
// from here on.
__device__ __forceinline__ void core_forbid(const IncBufs& b, int32_t v, int32_t c) {
  const int32_t w = (c - 1) >> 5;
  const uint32_t bit = 1u << ((c - 1) & 31);
  if (w == 0) {
    b.F[v] |= bit;
    return;
  }
  const int32_t w0 = b.fw_off[v];
  if (w <= b.fw_off[v + 1] - w0) b.Fx[w0 + w - 1] |= bit;  // (beyond: a color v can never take)
}

// Smallest color >= c that v's forbidden bitset does not hold.
__device__ __forceinline__ int32_t core_free_from(const IncBufs& b, int32_t v, int32_t c) {
  while (true) {
    const int32_t w = (c - 1) >> 5;
    const uint32_t rest = ~core_word(b, v, w) >> ((c - 1) & 31);
    if (rest) return c + __builtin_ctz(rest);
    c = 32 * (w + 1) + 1;
  }
}

// Bits of the forbidden colors [t, t + 64).
__device__ __forceinline__ uint64_t core_window(const IncBufs& b, int32_t v, int32_t t) {
  const int32_t w = (t - 1) >> 5, s = (t - 1) & 31;
  const uint64_t two = static_cast<uint64_t>(core_word(b, v, w + 1)) << 32 | core_word(b, v, w);
  return s ? two >> s | static_cast<uint64_t>(core_word(b, v, w + 2)) << (64 - s) : two;
}

// Smallest color > c that neither the window fw (of colors fb .. fb + 63) nor
// beyond it the bitset holds.
__device__ __forceinline__ int32_t core_next(const IncBufs& b, int32_t v, int32_t c, int32_t fb, uint64_t fw) {
  ++c;
  const int32_t d = c - fb;
  const uint64_t rest = d < 64 ? ~fw >> d : 0ull;
  return rest ? c + static_cast<int32_t>(__builtin_ctzll(rest)) : core_free_from(b, v, max(c, fb + 64));
}

__device__ __forceinline__ uint32_t core_key32(const KeySource& k, int32_t v) {
  if (k.rank) return ld_dev(&k.rank[v]);
  return fmix32((k.gid ? static_cast<uint32_t>(k.gid[v]) : static_cast<uint32_t>(v)) ^ k.hs);
}

}  // namespace

// Numbers the n worklist vertices by key, highest first: number = how many
// keys are higher (keys never tie).  order[number] = vertex, and the vertex's
// tentative-color entry holds its number until the rounds after this launch
// rewrite it (they write the tentative color of every worklist vertex before
// they read any).  Lane = key: a wavefront compares 64 keys with each of its
// vertices' and counts the ballot.  WIDE: 64-bit keys (explicit priorities,
// which may tie); else the hash or the degree rank decides alone.  Also clears
// the exchange words (round numbers start at 1).
template <bool WIDE>
__global__ __launch_bounds__(kCoreThreads) void core_rank_kernel(KeySource k, CoreWorklist q, int32_t n,
                                                                 int32_t* order, int32_t* T, uint64_t* words,
                                                                 int32_t num_words) {
  using Key = typename std::conditional<WIDE, uint64_t, uint32_t>::type;
  auto key = [&](int32_t v) -> Key {
    if constexpr (WIDE) return key_of(k, v);
    else return core_key32(k, v);
  };
  constexpr int V = kRankPer / kCoreWaves;
  __shared__ Key s_key[kRankChunk];
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int32_t i = blockIdx.x * kCoreThreads + tid; i < num_words; i += gridDim.x * kCoreThreads) words[i] = 0ull;
  const int32_t first = blockIdx.x * kRankPer + wave * V;
  Key kv[V];
  int32_t higher[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    kv[j] = first + j < n ? key(core_entry(q, first + j)) : 0;
    higher[j] = 0;
  }
  for (int32_t c0 = 0; c0 < n; c0 += kRankChunk) {
    const int32_t m = min(kRankChunk, n - c0);
    __syncthreads();
    for (int32_t e = tid; e < (m + kWave - 1) / kWave * kWave; e += kCoreThreads)
      s_key[e] = e < m ? key(core_entry(q, c0 + e)) : 0;  // 0 is above no key
    __syncthreads();
    for (int32_t e = lane; e < m; e += kWave) {
      const Key x = s_key[e];
#pragma unroll
      for (int j = 0; j < V; ++j) higher[j] += static_cast<int32_t>(__popcll(__ballot(x > kv[j])));
    }
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    if (first + j < n && lane == 0) {
      const int32_t v = core_entry(q, first + j);
      order[higher[j]] = v;
      T[v] = higher[j];
    }
  }
}

// Entries [0, all) of a vertex's active list (both parts) into its row of
// bits over the numbers, by `stride` threads from `first`, eight entries per
// thread in flight.  Entries that have committed are left out.
__device__ __forceinline__ void build_row(const IncBufs& b, const int32_t* lists, int split, int32_t v, int first,
                                          int stride, uint32_t* row) {
  constexpr int N = 8;
  const int32_t hlen = b.alen_in[v], llen = split ? b.llen[v] : 0;
  const int32_t* H = lists + b.aoff[v];
  const int32_t* Lo = lists + b.aoff[v + 1] - llen;
  const int32_t all = hlen + llen;
  for (int32_t e0 = first; e0 - first < all; e0 += N * stride) {
    int32_t u[N];
    bool live[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int32_t e = e0 + j * stride;
      u[j] = e < all ? (e < hlen ? H[e] : Lo[e - hlen]) : -1;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) live[j] = u[j] >= 0 && !((b.done[u[j] >> 5] >> (u[j] & 31)) & 1u);
#pragma unroll
    for (int j = 0; j < N; ++j) u[j] = live[j] ? b.T[u[j]] : 0;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (live[j]) atomicOr(&row[u[j] >> 5], 1u << (u[j] & 31));
  }
}

// A wavefront per vertex (its workgroup together for a list longer than
// kWaveList): the row, built in LDS; the tentative color; the forbidden colors
// from that on.  Bound by the chain list, committed bit, number.  (A workgroup
// per vertex, with two statistics atomics on one cache block each, took 263 us
// for 24576 vertices of RMAT scale 17.)
constexpr int32_t kWaveList = 2048;

__global__ __launch_bounds__(kBlock) void core_build_kernel(IncBufs b, CoreSet out, const int32_t* lists, int split,
                                                            int32_t stride, int32_t n) {
  __shared__ uint32_t s_rows[kWavesPerBlock][768];
  __shared__ int32_t s_long[kWavesPerBlock];  // the vertex if its list is long, else -1
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int32_t g = blockIdx.x * kWavesPerBlock + wave;
  uint32_t* s_row = s_rows[wave];
  for (int w = lane; w < stride; w += kWave) s_row[w] = 0u;
  if (lane == 0) s_long[wave] = -1;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (g < n) {
    const int32_t v = out.v[g];
    const int64_t all = static_cast<int64_t>(b.alen_in[v]) + (split ? b.llen[v] : 0);
    if (lane == 0) {
      const int32_t t = core_free_from(b, v, 1);
      out.t[g] = t;
      out.fw[g] = core_window(b, v, t);
      if (all > kWaveList) s_long[wave] = v;
    }
    if (all <= kWaveList) build_row(b, lists, split, v, lane, kWave, s_row);
  }
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < kWavesPerBlock; ++i)
    if (s_long[i] >= 0) build_row(b, lists, split, s_long[i], tid, kBlock, s_rows[i]);
  __syncthreads();
  if (g < n) {
    uint32_t* r = out.rows + static_cast<size_t>(g) * static_cast<size_t>(stride);
    for (int w = lane; w < stride; w += kWave) r[w] = s_row[w];
  }
  const int32_t base = blockIdx.x * kWavesPerBlock;
  if (base % kBlock == 0) {  // the statistics of kBlock vertices at once
    unsigned long long sum = 0;
    if (base + tid < n) {
      const int32_t x = out.v[base + tid];
      sum = static_cast<unsigned long long>(b.alen_in[x]) + static_cast<unsigned long long>(split ? b.llen[x] : 0);
    }
    // list entry, committed bits, number; the row
    unsigned long long bytes = sum ? 12ull * sum + 4ull * static_cast<unsigned long long>(stride) : 0ull;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      sum += __shfl_xor(sum, off, kWave);
      bytes += __shfl_xor(bytes, off, kWave);
    }
    if (lane_id() == 0 && sum) {
      atomicAdd(&acc_slot(b.acc)[2], sum);
      atomicAdd(&acc_slot(b.acc)[7], bytes);
    }
  }
}

namespace {

enum CoreEnd : int { kCoreDone, kCoreCapped, kCoreSpread, kCoreFail, kCoreHandOver };

// Shared values of a stage over several workgroups.
template <int U, int NT>
struct CoreShared {
  int32_t v[32 * U];      // vertex, -1: none
  int32_t t[32 * U];      // tentative (then committed) color
  int32_t won[32 * U];    // round it committed in, 0: not yet
  int32_t fb[32 * U];     // forbidden colors: bit d of fw stands for color fb + d, t - 32 <= fb <= t
  uint64_t fw[32 * U];
  uint32_t hit[kCoreSlots][U];  // phase B: the vertices with a neighbour that committed the slot's color
  uint32_t slots[U];
  uint32_t near_row[32 * U][U];      // higher-key neighbours inside the workgroup
  uint32_t near_bits[kCoreSlots][U]; // phase A's words of the workgroup itself
  int32_t gmin[2], gmax[2], total[2];
  int32_t fail;
  int32_t scan[16];
  uint32_t live[768];                // hand-over: the vertices left, and how many precede each word
  int32_t before[768];
  uint32_t pack[NT / kWave][kMidMax / 32];
};

// Waits for word w's round `tag` in every slot of `slots` and gives each to
// take(slot, bits); with a summary word `sum`, waits for that too (*payload
// receives its lower half).  D words are in flight at a time, the summary word
// among the first.  Returns false after `deadline` clock ticks.
template <int D, typename F>
__device__ __forceinline__ bool core_fetch(const uint64_t* x, uint32_t slots, int32_t W, int32_t w, uint32_t tag,
                                           const uint64_t* sum, uint32_t* payload, uint64_t deadline, F&& take) {
  bool more = sum != nullptr;
  while (slots || more) {
    int s[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      s[j] = slots ? __builtin_ctz(slots) : -1;
      slots &= slots - 1u;
    }
    uint64_t y[D], z = 0;
    uint64_t t0 = 0;
    for (int spin = 0;; ++spin) {
      if (more) z = ld_dev(sum);
#pragma unroll
      for (int j = 0; j < D; ++j) y[j] = s[j] >= 0 ? ld_dev(&x[s[j] * W + w]) : 0ull;
      bool ready = !more || static_cast<uint32_t>(z >> 32) == tag;
#pragma unroll
      for (int j = 0; j < D; ++j) ready = ready && (s[j] < 0 || static_cast<uint32_t>(y[j] >> 32) == tag);
      if (ready) break;
      if (spin >= 64) {
        __builtin_amdgcn_s_sleep(1);
        const uint64_t now = static_cast<uint64_t>(wall_clock64());
        if (t0 == 0) t0 = now;
        else if (now - t0 > deadline) return false;
      }
    }
    if (more) *payload = static_cast<uint32_t>(z);
    more = false;
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (s[j] >= 0) take(s[j], static_cast<uint32_t>(y[j]));
  }
  return true;
}

// Wavefront reduction without LDS (row shifts, then row broadcasts): the
// result of all 64 lanes.
template <typename F>
__device__ __forceinline__ int32_t wave_reduce(int32_t x, int32_t none, F&& f) {
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x111, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x112, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x114, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x118, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x142, 0xa, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(none, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, kWave - 1);
}

// The slots of colors lo .. hi (hi - lo < kCoreSlots).
__device__ __forceinline__ uint32_t core_slots(int32_t lo, int32_t hi) {
  if (lo > hi) return 0u;
  const uint32_t span = static_cast<uint32_t>(hi - lo);
  const uint32_t ones = span >= 31u ? ~0u : (1u << (span + 1u)) - 1u;
  const int s = lo & (kCoreSlots - 1);
  return s ? (ones << s) | (ones >> (32 - s)) : ones;
}

// Adds what one vertex of a stage contributes at the stage's end: its color
// if it committed, its rounds (a worklist entry and its work each) and the
// largest color.  Called by whole wavefronts; v < 0: nothing.
__device__ __forceinline__ void core_account(const IncBufs& b, int32_t v, int32_t t, int32_t won, int round0, int last) {
  unsigned long long rounds = 0, work = 0;
  int32_t maxc = 0;
  if (v >= 0) {
    rounds = static_cast<unsigned long long>((won ? won : last) - round0 + 1);
    work = rounds * static_cast<unsigned long long>(b.work[v]);
    if (won) {
      st_dev(&b.C[v], t);
      maxc = t;
    }
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    rounds += __shfl_xor(rounds, o, kWave);
    work += __shfl_xor(work, o, kWave);
    maxc = max(maxc, __shfl_xor(maxc, o, kWave));
  }
  if (lane_id() == 0) {
    if (rounds) atomicAdd(&acc_slot(b.acc)[0], rounds);
    if (work) atomicAdd(&acc_slot(b.acc)[1], work);
    if (maxc > 0) atomicMax(b.maxc, maxc);
  }
}

// Word of lane `lane`'s q-th register: four (two) consecutive words per lane,
// so that a slot mask is read 16 (8) bytes at a time.
template <int K>
__device__ __forceinline__ int core_word_of(int lane, int q) {
  constexpr int B = K < 4 ? K : 4;
  return (q / B) * (kWave * B) + lane * B + q % B;
}

// One stage of several workgroups over n vertices from round r on, until at
// most stop_at are left.  U: 32-bit row words (32 vertices each) a workgroup
// of NT threads owns; K: row words per lane; the stage's first ceil(n / 32 U)
// workgroups take part.
//
// Bound by the two exchanges (publish, wait, read: 3.5-5 us each with 256
// workgroups, about 2 us with 64) and the detect's LDS reads (3 us).  A round
// takes 14-18 us with 256 workgroups and 7 us with 64; with the committed bits
// of every color in use read in phase B and every loser's row tested against
// them, 25-30 and 8.5 us.
template <int U, int K, int NT>
__device__ __forceinline__ CoreEnd core_stage(const IncBufs& b, const CoreSet& in, const CoreExchange& x,
                                              const CoreSet& out, int32_t n, int32_t stop_at, int& r, int round_cap,
                                              uint32_t* s_mask, CoreShared<U, NT>& sh, int32_t* left_n,
                                              uint64_t deadline) {
  constexpr int P = 32 * U;            // vertices of the workgroup
  constexpr int V = P / (NT / kWave);  // vertices of a wavefront
  constexpr int S = kWave * K;         // row words; those from W on are zero
  constexpr int B = K < 4 ? K : 4;
  constexpr int D = K < 4 ? 4 : 8;     // exchange words in flight per thread
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // consecutive vertices on one XCD (workgroups go round the eight), as they
  // read the same cache lines of a committed vertex's row
  const int32_t blocks = (n + P - 1) / P;
  const int32_t xcd = static_cast<int32_t>(blockIdx.x) % 8;
  const int32_t blk = xcd * (blocks / 8) + min(xcd, blocks % 8) + static_cast<int32_t>(blockIdx.x) / 8;
  const int32_t W = U * blocks;
  const int round0 = r;

  if (tid < P) {
    const int32_t g = blk * P + tid;
    const bool have = g < n;
    sh.v[tid] = have ? ld_dev(&in.v[g]) : -1;
    sh.t[tid] = sh.fb[tid] = have ? ld_dev(&in.t[g]) : 1;
    sh.fw[tid] = have ? ld_dev(&in.fw[g]) : 0ull;
    sh.won[tid] = 0;
  }
  if (tid < 2) {
    sh.gmin[tid] = INT_MAX;
    sh.gmax[tid] = 0;
    sh.total[tid] = 0;
  }
  if (tid == 0) sh.fail = 0;
  // the wavefront's rows.  The part of a row inside the workgroup is kept
  // apart as well, below the vertex's own bit only: the rest of phase A's
  // test then needs no limit
  uint32_t row[V][K];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const int32_t g = blk * P + wave * V + j;
    const uint32_t* src = in.rows + static_cast<size_t>(g) * S;
#pragma unroll
    for (int q = 0; q < K; q += 2) {
      const uint64_t y = g < n ? ld_dev(reinterpret_cast<const uint64_t*>(src + core_word_of<K>(lane, q))) : 0ull;
      row[j][q] = static_cast<uint32_t>(y);
      row[j][q + 1] = static_cast<uint32_t>(y >> 32);
    }
  }
  for (int q = tid; q < P * U; q += NT) {
    const int i = q / U, u = q % U;
    const int32_t g = blk * P + i;
    const uint32_t y = g < n ? ld_dev(&in.rows[static_cast<size_t>(g) * S + blk * U + u]) : 0u;
    sh.near_row[i][u] = u < i / 32 ? y : u == i / 32 ? y & ((1u << (i & 31)) - 1u) : 0u;
  }
  __syncthreads();

  // the wavefront's vertices (uniform over its lanes)
  int32_t t[V];
  uint32_t act = 0;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    t[j] = __builtin_amdgcn_readfirstlane(sh.t[wave * V + j]);
    act |= __builtin_amdgcn_readfirstlane(sh.v[wave * V + j]) >= 0 ? 1u << j : 0u;
  }
  // exchange reads: this thread takes the words rw, rw + NT, ... of the slots
  // s with s mod subs = rs
  int32_t wp = 32;
  while (wp < W && wp < NT) wp <<= 1;
  const int32_t subs = NT / wp, rs = tid / wp;
  uint32_t mine = 0;
  for (int s = 0; s < kCoreSlots; ++s) mine |= (s % subs) == rs ? 1u << s : 0u;
  const int32_t my_word = blk * U + wave;  // published by wavefronts 0 .. U-1
  int32_t gmin = 0, gmax = 0;
  uint64_t bytes_a = 0;
  uint32_t seen = 0;  // committed vertices whose rows this thread read
  CoreEnd end = kCoreDone;
  for (;; ++r) {
    const uint32_t tag = static_cast<uint32_t>(r);
    const uint64_t hi = static_cast<uint64_t>(tag) << 32;
    const int par = r & 1;
    // ---- phase A: the bits of every color in use
    if (wave < U) {
      const int i = 32 * wave + (lane & 31);
      const bool on = lane < 32 && sh.v[i] >= 0 && sh.won[i] == 0;
      const int32_t ti = sh.t[i];
      uint64_t rem = __ballot(on);
      const uint32_t count = static_cast<uint32_t>(__popcll(rem));
      uint32_t val = 0, slots = 0;
      int32_t mn = INT_MAX, mx = 0;
      while (rem) {
        const int32_t c = __builtin_amdgcn_readlane(ti, static_cast<int>(__builtin_ctzll(rem)));
        const uint64_t m = __ballot(on && ti == c);
        if (lane == (c & (kCoreSlots - 1))) val |= static_cast<uint32_t>(m);
        slots |= 1u << (c & (kCoreSlots - 1));
        mn = min(mn, c);
        mx = max(mx, c);
        rem &= ~m;
      }
      if (lane < 32) {
        st_dev(&x.A[lane * W + my_word], hi | val);
        sh.near_bits[lane][wave] = val;
      }
      if (lane == 32) {
        // summary: count (6 bits), smallest color (20), span (6; 63: too wide)
        const bool wide = count && (mx - mn >= kCoreSlots || mx >= kCoreMaxColor);
        const uint32_t p = count | (count ? (wide ? 0u : static_cast<uint32_t>(mn)) << 6 : 0u) |
                           (count ? (wide ? 63u : static_cast<uint32_t>(mx - mn)) << 26 : 0u);
        st_dev(&x.ma[my_word], hi | p);
        sh.slots[wave] = slots;
      }
    }
    __syncthreads();
    uint32_t slots = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) slots |= sh.slots[u];
    // only higher keys matter: the words below the workgroup's own
    int32_t cnt = 0, mn = INT_MAX, mx = 0;
    for (int32_t rw = tid & (wp - 1); rw < W; rw += wp) {
      const bool below = rw < blk * U;
      uint32_t p = 0;
      if (!core_fetch<D>(x.A, below ? slots & mine : 0u, W, rw, tag, rs == 0 ? &x.ma[rw] : nullptr, &p, deadline,
                         [&](int s, uint32_t y) { s_mask[s * S + rw] = y; }))
        sh.fail = 1;
      if (!below)
        for (uint32_t z = slots & mine; z; z &= z - 1u) s_mask[__builtin_ctz(z) * S + rw] = 0u;
      if ((p & 63u) != 0u) {
        const int32_t c = static_cast<int32_t>((p >> 6) & 0xFFFFFu);
        cnt += static_cast<int32_t>(p & 63u);
        mn = min(mn, c);
        mx = max(mx, c + static_cast<int32_t>(p >> 26));
      }
    }
    if (wave * kWave < wp) {
      cnt = wave_reduce(cnt, 0, [](int32_t a, int32_t c) { return a + c; });
      mn = wave_reduce(mn, INT_MAX, [](int32_t a, int32_t c) { return min(a, c); });
      mx = wave_reduce(mx, 0, [](int32_t a, int32_t c) { return max(a, c); });
      if (lane == 0 && cnt) {
        atomicAdd(&sh.total[par], cnt);
        atomicMin(&sh.gmin[par], mn);
        atomicMax(&sh.gmax[par], mx);
      }
    }
    __syncthreads();
    const int32_t total = __builtin_amdgcn_readfirstlane(sh.total[par]);
    gmin = __builtin_amdgcn_readfirstlane(sh.gmin[par]);
    gmax = __builtin_amdgcn_readfirstlane(sh.gmax[par]);
    if (sh.fail) {
      end = kCoreFail;
      break;
    }
    if (total == 0) break;
    if (r > round_cap) {
      end = kCoreCapped;
      break;
    }
    // (a stage whose colors are about to outgrow the slots keeps its vertices:
    // as long as no stage has written, the rounds can still go elsewhere; the
    // one-workgroup stage takes any spread)
    if (total <= stop_at && (stop_at == kSmallMax || gmax - gmin < kCoreSlots * 3 / 4)) {
      // the vertices left: every slot's bits of every word
      for (int32_t w = tid; w < W; w += NT) {
        uint32_t y = 0;
        if (!core_fetch<D>(x.A, gmax - gmin >= kCoreSlots ? ~0u : core_slots(gmin, gmax), W, w, tag, nullptr, nullptr,
                           deadline, [&](int, uint32_t z) { y |= z; }))
          sh.fail = 1;
        sh.live[w] = y;
      }
      __syncthreads();
      if (sh.fail) {
        end = kCoreFail;
        break;
      }
      // vertices left before each word: by blocks of 64 words, then over these
      for (int32_t w0 = wave * kWave; w0 < W; w0 += NT) {
        const int32_t w = w0 + lane;
        const int32_t c = w < W ? static_cast<int32_t>(__popc(sh.live[w])) : 0;
        int32_t incl = c;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
          const int32_t y = __shfl_up(incl, o, kWave);
          if (lane >= o) incl += y;
        }
        if (lane == kWave - 1) sh.scan[w0 / kWave] = incl;
        if (w < W) sh.before[w] = incl - c;
      }
      __syncthreads();
      for (int32_t w = tid; w < W; w += NT) {
        int32_t add = 0;
        for (int o = 0; o < w / kWave; ++o) add += sh.scan[o];
        sh.before[w] += add;
      }
      __syncthreads();
      const int32_t stride = row_words(stop_at);
#pragma unroll 1
      for (int i = wave * V; i < wave * V + V; ++i) {
        if (sh.v[i] < 0 || sh.won[i] != 0) continue;
        const int32_t own = blk * U + i / 32, ti = sh.t[i];
        const int32_t me = sh.before[own] + static_cast<int32_t>(__popc(sh.live[own] & ((1u << (i & 31)) - 1u)));
        const uint32_t* src = in.rows + static_cast<size_t>(blk * P + i) * S;
        // its forbidden colors: the bitset's, and those its neighbours
        // committed in the core stages
        const int32_t ahead = ti - sh.fb[i];
        const uint64_t fw = core_window(b, sh.v[i], ti) | (ahead < 64 ? sh.fw[i] >> ahead : 0ull);
        // its row over the vertices left
        uint32_t* p = sh.pack[wave];
        for (int w = lane; w < stride; w += kWave) p[w] = 0u;
        wave_step();
        for (int w = lane; w < W; w += kWave) {
          const uint32_t live = sh.live[w];
          for (uint32_t z = ld_dev(&src[w]) & live; z; z &= z - 1u) {
            const int32_t g = sh.before[w] + static_cast<int32_t>(__popc(live & ((z & (0u - z)) - 1u)));
            atomicOr(&p[g >> 5], 1u << (g & 31));
          }
        }
        wave_step();
        uint32_t* dst = out.rows + static_cast<size_t>(me) * stride;
        for (int w = lane; w < stride; w += kWave) st_dev(&dst[w], p[w]);
        wave_step();
        if (lane == 0) {
          st_dev(&out.v[me], sh.v[i]);
          st_dev(&out.t[me], ti);
          st_dev(&out.fw[me], fw);
        }
      }
      *left_n = total;
      end = kCoreHandOver;
      break;
    }
    if (gmax - gmin >= kCoreSlots) {
      end = kCoreSpread;
      break;
    }
    if (blk == 0 && tid == 0) {
      const int gr = r + b.round_base;
      if (b.trace && gr <= b.trace_cap) st_dev(&b.trace[gr - 1], total);
    }
    bytes_a += 8ull * static_cast<uint64_t>(W + U * kCoreSlots) +
               8ull * static_cast<uint64_t>(__popc(slots)) * static_cast<uint64_t>(blk * U);
    if (tid == 0) {
      sh.total[par ^ 1] = 0;
      sh.gmin[par ^ 1] = INT_MAX;
      sh.gmax[par ^ 1] = 0;
    }
    for (int q = tid; q < kCoreSlots * U; q += NT) sh.hit[q / U][q % U] = 0u;
    // ---- detect: a vertex of higher key with the same tentative color
    // (two vertices at a time, so that their reads overlap)
#pragma unroll
    for (int j = 0; j < V; j += 2) {
      const uint32_t two = (act >> j) & 3u;
      if (two == 0u) continue;
      uint32_t hit[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int slot = t[j + h] & (kCoreSlots - 1);
        hit[h] = lane < U ? sh.near_row[wave * V + j + h][lane] & sh.near_bits[slot][lane] : 0u;
        const uint32_t* m = s_mask + slot * S + lane * B;
#pragma unroll
        for (int q = 0; q < K; ++q) hit[h] |= row[j + h][q] & m[(q / B) * (kWave * B) + q % B];
      }
      uint32_t lost = __ballot(hit[0] != 0u) != 0ull ? 1u : 0u;
      lost |= __ballot(hit[1] != 0u) != 0ull ? 2u : 0u;
      const uint32_t wins = two & ~lost;
      act &= ~(wins << j);
      if (lane < 2 && (wins >> lane) & 1u) sh.won[wave * V + j + lane] = r;
    }
    __syncthreads();
    // ---- phase B: the vertices that committed and their colors' slots
    if (wave < U) {
      const int i = 32 * wave + (lane & 31);
      const int32_t ti = sh.t[i];
      const uint64_t m = __ballot(lane < 32 && sh.won[i] == r);
      uint32_t val = 0;
      int k = 0;
      for (uint64_t z = m; z; z &= z - 1ull, ++k) {
        const uint32_t c = static_cast<uint32_t>(__builtin_amdgcn_readlane(ti, static_cast<int>(__builtin_ctzll(z))));
        if (lane == k / kCoreColors) val |= (c & (kCoreSlots - 1)) << (5 * (k % kCoreColors));
      }
      if (lane == 0 || (lane < kCoreColorWords && lane * kCoreColors < k)) st_dev(&x.B[lane * W + my_word], hi | val);
      if (lane == 32) st_dev(&x.mb[my_word], hi | static_cast<uint32_t>(m));
    }
    constexpr int R = (S + NT - 1) / NT;  // words per thread
    static_assert(R <= 2, "the word loop picks the first or the last");
    uint32_t won_bits[R], colors[R];
    {
      uint64_t t0 = 0;
      for (int spin = 0;; ++spin) {
        uint64_t z[R], y[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const int32_t rw = tid + i * NT;
          z[i] = rw < W ? ld_dev(&x.mb[rw]) : hi;
          y[i] = rw < W ? ld_dev(&x.B[rw]) : hi;
        }
        bool ready = true;
#pragma unroll
        for (int i = 0; i < R; ++i) {
          ready = ready && static_cast<uint32_t>(z[i] >> 32) == tag && static_cast<uint32_t>(y[i] >> 32) == tag;
          won_bits[i] = static_cast<uint32_t>(z[i]);
          colors[i] = static_cast<uint32_t>(y[i]);
        }
        if (ready) break;
        if (spin >= 64) {
          __builtin_amdgcn_s_sleep(1);
          const uint64_t now = static_cast<uint64_t>(wall_clock64());
          if (t0 == 0) t0 = now;
          else if (now - t0 > deadline) {
            sh.fail = 1;
#pragma unroll
            for (int i = 0; i < R; ++i) won_bits[i] = 0;
            break;
          }
        }
      }
    }
    // Each committed vertex's neighbours here, its row's words of the
    // workgroup's own vertices, are added to the neighbours of its color.
#pragma unroll 1
    for (int i = 0; i < R; ++i) {
      uint32_t bits = i == 0 ? won_bits[0] : won_bits[R - 1];
      if (bits == 0u) continue;
      const int32_t rw = tid + i * NT;
      const int count = __popc(bits);
      uint32_t more[kCoreColorWords - 1] = {};  // the colors beyond the first word's
      if (count > kCoreColors) {
        uint64_t t0 = 0;
        for (int spin = 0;; ++spin) {
          bool ready = true;
#pragma unroll
          for (int q = 1; q < kCoreColorWords; ++q) {
            const uint64_t y = q * kCoreColors < count ? ld_dev(&x.B[q * W + rw]) : hi;
            ready = ready && static_cast<uint32_t>(y >> 32) == tag;
            more[q - 1] = static_cast<uint32_t>(y);
          }
          if (ready) break;
          if (spin >= 64) {
            __builtin_amdgcn_s_sleep(1);
            const uint64_t now = static_cast<uint64_t>(wall_clock64());
            if (t0 == 0) t0 = now;
            else if (now - t0 > deadline) {
              sh.fail = 1;
              break;
            }
          }
        }
      }
      uint32_t packed = i == 0 ? colors[0] : colors[R - 1];
      int left = kCoreColors;  // colors left in packed
      while (bits) {
        // N at a time, so that their reads overlap
        constexpr int N = 4;
        uint32_t own[N][U];
        int32_t slot[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
#pragma unroll
          for (int u = 0; u < U; ++u) own[j][u] = 0u;
          slot[j] = 0;
          if (bits == 0u) continue;
          const uint32_t* src = in.rows + static_cast<size_t>(32 * rw + __builtin_ctz(bits)) * S + blk * U;
#pragma unroll
          for (int u = 0; u < U; ++u) own[j][u] = src[u];
          bits &= bits - 1u;
          if (left == 0) {
            packed = more[0];
#pragma unroll
            for (int q = 0; q + 1 < kCoreColorWords - 1; ++q) more[q] = more[q + 1];
            left = kCoreColors;
          }
          slot[j] = static_cast<int32_t>(packed & 31u);
          packed >>= 5;
          --left;
        }
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (own[j][u]) atomicOr(&sh.hit[slot[j]][u], own[j][u]);
      }
      seen += static_cast<uint32_t>(count);
    }
    __syncthreads();
    if (sh.fail) {
      end = kCoreFail;
      break;
    }
    // ---- the losers' next first fit
    if (tid < P && sh.v[tid] >= 0 && sh.won[tid] == 0) {
      const int32_t c = sh.t[tid], fb = sh.fb[tid];
      uint64_t fw = sh.fw[tid];
      uint32_t add = 0;  // bit d: a neighbour has committed color c + d in this round
      for (int32_t y = c; y <= gmax; ++y) add |= ((sh.hit[y & (kCoreSlots - 1)][tid / 32] >> (tid & 31)) & 1u) << (y - c);
      if (add) {
        fw |= static_cast<uint64_t>(add) << (c - fb);
        sh.fw[tid] = fw;
      }
      const uint64_t rest = ~fw >> (c - fb);
      const int32_t next = rest ? c + static_cast<int32_t>(__builtin_ctzll(rest)) : core_free_from(b, sh.v[tid], fb + 64);
      if (next != c) {
        sh.t[tid] = next;
        const int32_t ahead = next - fb;
        if (ahead > 32) {  // the window goes on from here
          sh.fb[tid] = next;
          sh.fw[tid] = (ahead < 64 ? fw >> ahead : 0ull) | core_window(b, sh.v[tid], next);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < V; ++j) t[j] = __builtin_amdgcn_readfirstlane(sh.t[wave * V + j]);
  }
  if (end != kCoreFail && end != kCoreSpread) {
    if (wave * kWave < P) {
      const bool have = tid < P;
      core_account(b, have ? sh.v[tid] : -1, have ? sh.t[tid] : 0, have ? sh.won[tid] : 0, round0, r - 1);
    }
    const int32_t rows = wave_reduce(static_cast<int32_t>(seen), 0, [](int32_t p, int32_t q) { return p + q; });
    if (lane == 0 && rows) atomicAdd(&acc_slot(b.acc)[7], 4ull * U * static_cast<unsigned long long>(rows));
    if (tid == 0) {
      atomicAdd(&acc_slot(b.acc)[6], static_cast<unsigned long long>(bytes_a));
      atomicAdd(&acc_slot(b.acc)[7], 16ull * static_cast<unsigned long long>(W) * static_cast<unsigned long long>(r - round0));
    }
  }
  return end;
}

struct SmallShared {
  // phase A: bits of the tentative colors; phase B: committed bits, in a slot
  // per lane (rows padded so that neighbouring slots start on other banks)
  alignas(16) uint64_t a[kCoreSlots][kCoreWaves + 2];
  alignas(16) uint64_t c[kWave][kCoreWaves + 2];
  alignas(16) uint64_t w[kCoreWaves];      // phase B without slots: commits to take in
  int32_t t[kSmallMax];                    // tentative color, or minus the committed one
  int32_t gmin[2], gmax[2], total[2];
};

// The one-workgroup stage: a thread per vertex, its row of 1024 bits in
// registers, the slot masks in LDS.  While the tentative colors span at most
// kCoreSlots, a slot holds one color; beyond, the colors that share the slot
// are told apart by the entries of sh.t that the row meets in it.
//
// What the stage's vertices have committed is in slots too (fw and the bitset
// hold what was committed before), and a loser tests every color it steps
// over up to `top`, the largest tentative color of any round so far: no
// committed color of the stage is above it.  The largest tentative color of
// the round will not do, as it falls when its holders commit.  The committed
// colors that still matter, gmin .. top, have a slot each while they span at
// most kWave colors (a slot is cleared when its color has fallen below gmin,
// which never falls itself).  In rounds beyond that every loser takes its
// neighbours' new commits into its window, or past that into its own bitset,
// instead.  (1000 vertices of mean degree 800 over 300 initial colors, 53
// rounds: 1.2 ms a call; with the colors of the whole row compared for every
// step 63 ms, in the tail kernel 1.9 ms.)
__device__ __forceinline__ CoreEnd core_small(const IncBufs& b, const CoreSet& in, int32_t n, int& r, int round_cap,
                                              SmallShared& sh) {
  constexpr int R = kSmallMax / 64;
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int round0 = r;
  const bool have = tid < n;
  const int32_t v = have ? ld_dev(&in.v[tid]) : -1;
  int32_t t = have ? ld_dev(&in.t[tid]) : 1;
  const int32_t fb = t;
  uint64_t fw = have ? ld_dev(&in.fw[tid]) : 0ull;
  uint64_t row[R], near = 0;
#pragma unroll
  for (int p = 0; p < R; ++p) {
    row[p] = have ? ld_dev(reinterpret_cast<const uint64_t*>(in.rows + static_cast<size_t>(tid) * (2 * R)) + p) : 0ull;
    if (p == wave) near = row[p] & ((1ull << lane) - 1ull);
  }
  if (tid < 2) {
    sh.gmin[tid] = INT_MAX;
    sh.gmax[tid] = 0;
    sh.total[tid] = 0;
  }
  int32_t won = 0;
  bool act = have;
  uint64_t comm = 0;
  int32_t comm_c = 0;
  bool comm_ok = true;  // comm holds every commit so far of the colors it stands for
  bool fw_ok = true;    // the losers' windows and bitsets hold every commit so far
  int32_t top = 0;
  CoreEnd end = kCoreDone;
  __syncthreads();
  for (;; ++r) {
    const int par = r & 1;
    // ---- phase A
    const uint64_t on = __ballot(act);
    {
      uint64_t rem = on, val = 0;
      int32_t mn = INT_MAX, mx = 0;
      while (rem) {
        const int32_t c = __builtin_amdgcn_readlane(t, static_cast<int>(__builtin_ctzll(rem)));
        const uint64_t m = __ballot(act && t == c);
        if (lane == (c & (kCoreSlots - 1))) val |= m;
        mn = min(mn, c);
        mx = max(mx, c);
        rem &= ~m;
      }
      if (lane < kCoreSlots) sh.a[lane][wave] = val;
      if (lane == 0 && on) {
        atomicAdd(&sh.total[par], static_cast<int32_t>(__popcll(on)));
        atomicMin(&sh.gmin[par], mn);
        atomicMax(&sh.gmax[par], mx);
      }
      sh.t[tid] = act ? t : won ? -t : 0;
    }
    __syncthreads();
    const int32_t total = __builtin_amdgcn_readfirstlane(sh.total[par]);
    const int32_t gmin = __builtin_amdgcn_readfirstlane(sh.gmin[par]);
    const int32_t gmax = __builtin_amdgcn_readfirstlane(sh.gmax[par]);
    if (total == 0) break;
    if (r > round_cap) {
      end = kCoreCapped;
      break;
    }
    if (tid == 0) {
      const int gr = r + b.round_base;
      if (b.trace && gr <= b.trace_cap) st_dev(&b.trace[gr - 1], total);
      // for the next round's phase A, which other wavefronts may reach as
      // soon as they have passed this round's second barrier
      sh.total[par ^ 1] = 0;
      sh.gmin[par ^ 1] = INT_MAX;
      sh.gmax[par ^ 1] = 0;
    }
    const bool fast = gmax - gmin < kCoreSlots;
    top = max(top, gmax);
    const bool slots = top - gmin < kWave;
    // ---- detect
    bool wins = false;
    if (on) {
      bool hit = false;
      const uint64_t* m = sh.a[t & (kCoreSlots - 1)];
      if (fast) {
        uint64_t y = near & m[wave];
#pragma unroll
        for (int p = 0; p < R; ++p)
          if (p < wave) y |= row[p] & m[p];
        hit = y != 0ull;
      } else if (act) {
#pragma unroll
        for (int p = 0; p < R; ++p)
          for (uint64_t y = (p < wave ? row[p] : p == wave ? near : 0ull) & m[p]; y && !hit; y &= y - 1ull)
            hit = sh.t[64 * p + __builtin_ctzll(y)] == t;
      }
      wins = act && !hit;
    }
    if (!fast) __syncthreads();  // every tentative color has been read
    // ---- phase B
    const uint64_t ws = __ballot(wins);
    if (wins) {
      act = false;
      won = r;
      if (!slots) sh.t[tid] = -t;
    }
    if (slots) {
      const int32_t c = gmin + ((lane - gmin) & (kWave - 1));
      if (!comm_ok) {  // rounds without slots came before: count afresh
        comm = 0;
        for (int s = 0; s < kWave; ++s) {
          const int32_t cs = gmin + ((s - gmin) & (kWave - 1));
          const uint64_t m = __ballot(won != 0 && t == cs);
          if (lane == s) comm = m;
        }
      } else {
        if (comm_c != c) comm = 0;
        uint64_t rem = ws;
        while (rem) {
          const int32_t cw = __builtin_amdgcn_readlane(t, static_cast<int>(__builtin_ctzll(rem)));
          const uint64_t m = __ballot(wins && t == cw);
          if (lane == (cw & (kWave - 1))) comm |= m;
          rem &= ~m;
        }
      }
      comm_c = c;
      sh.c[lane][wave] = comm;
    } else {
      // rounds with slots came before: their commits as well
      const uint64_t all = __ballot(won != 0);
      if (lane == 0) sh.w[wave] = fw_ok ? ws : all;
    }
    comm_ok = slots;
    fw_ok = !slots;
    __syncthreads();
    // ---- next first fit
    if (act && slots) {
      while (t <= top) {
        const uint64_t* m = sh.c[t & (kWave - 1)];
        uint64_t y = 0;
#pragma unroll
        for (int p = 0; p < R; ++p) y |= row[p] & m[p];
        if (y == 0ull) break;
        t = core_next(b, v, t, fb, fw);
      }
    } else if (act) {
      uint64_t y[R];
#pragma unroll
      for (int p = 0; p < R; ++p) y[p] = row[p] & sh.w[p];
#pragma unroll
      for (int p = 0; p < R; ++p) {
        for (; y[p]; y[p] &= y[p] - 1ull) {
          const int32_t c = -sh.t[64 * p + __builtin_ctzll(y[p])];
          if (c < t) continue;
          if (c - fb < 64) fw |= 1ull << (c - fb);
          else core_forbid(b, v, c);
        }
      }
      t = core_next(b, v, t - 1, fb, fw);
    }
    if (!slots) __syncthreads();  // every committed color has been read
  }
  core_account(b, v, t, won, round0, r - 1);
  if (tid == 0) atomicAdd(&acc_slot(b.acc)[7], static_cast<unsigned long long>(n) * (4ull * row_words(kSmallMax) + 20ull));
  return end;
}

// Hand-over between two stages: the workgroup's stores are done, and the next
// stage's workgroups wait for every workgroup of the one before.
__device__ __forceinline__ void core_hand_over(uint64_t* flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&flag[blockIdx.x], 1ull << 32, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool core_take_over(const uint64_t* flag, int32_t blocks, uint64_t deadline, int32_t* s_ok) {
  if (threadIdx.x == 0) *s_ok = 1;
  __syncthreads();
  uint32_t p;
  if (static_cast<int32_t>(threadIdx.x) < blocks &&
      !core_fetch<1>(flag, 0u, 0, 0, 1u, &flag[threadIdx.x], &p, deadline, [](int, uint32_t) {}))
    *s_ok = 0;
  __syncthreads();
  return *s_ok != 0;
}

}  // namespace

// How the wide stage ended, for the launch after it.
struct CoreHeader {
  int32_t handed;  // 1: set 1 holds the vertices left
  int32_t left;    // how many
  int32_t round;   // the round to go on from
  int32_t pad;
};

// Rounds from round0 on over the n > kMidMax vertices of set 0, until at most
// kMidMax are left in set 1.
template <int U, int K, int NT>
__global__ __launch_bounds__(NT) void core_wide_kernel(IncBufs b, CoreSet in, CoreExchange x, CoreSet out,
                                                       CoreHeader* head, int32_t n, int round0, int round_cap,
                                                       uint32_t* bar, int32_t* err, int32_t* left, uint64_t deadline,
                                                       uint64_t checkin_ticks) {
  __shared__ alignas(16) uint32_t s_mask[kCoreSlots * kWave * K];
  __shared__ CoreShared<U, NT> sh;
  __shared__ int32_t s_ok;
  if (!tail_checkin(&bar[kBarCheckin], &bar[kBarState], err, checkin_ticks, &s_ok)) return;
  int r = round0;
  int32_t m = n;
  const CoreEnd end = core_stage<U, K, NT>(b, in, x, out, n, kMidMax, r, round_cap, s_mask, sh, &m, deadline);
  if (threadIdx.x != 0) return;
  if (end == kCoreFail) {
    atomicOr(err, kErrTailBarrier);
  } else if (blockIdx.x == 0) {
    if (end == kCoreSpread) {
      atomicOr(err, kErrCoreWindow);
    } else if (end == kCoreHandOver) {
      atomicOr(err, kErrCoreHanded);
      head->left = m;
      head->round = r;
      head->handed = 1;
    } else {
      atomicMax(b.rounds_done, r - 1 + b.round_base);
      if (end == kCoreCapped) st_dev(left, 1);
    }
  }
}

// The rounds over at most kMidMax vertices: set 0's n vertices from round0
// on, or (head) what the wide stage left in set 1.
__global__ __launch_bounds__(kCoreThreads) void core_kernel(IncBufs b, CoreScratch x, const CoreHeader* head, int32_t n,
                                                            int round0, int round_cap, uint32_t* bar, int32_t* err,
                                                            int32_t* left, uint64_t deadline, uint64_t checkin_ticks) {
  __shared__ alignas(16) uint32_t s_mask[kCoreSlots * kWave * 2];
  __shared__ union {
    CoreShared<2, kCoreThreads> mid;
    SmallShared small;
  } sh;
  __shared__ int32_t s_ok;
  if (head) {
    // (a workgroup whose wait gave up has not written its part of set 1)
    if (!head->handed || (ld_dev(err) & kErrTailBarrier)) return;
    n = head->left;
    round0 = head->round;
  }
  // (a second launch of the call: check-in words of its own)
  if (!tail_checkin(&bar[head ? kBarGroup : kBarCheckin], &bar[head ? kBarGroup + 32 : kBarState], err, checkin_ticks,
                    &s_ok))
    return;
  const int32_t blocks = (n + 63) / 64;
  if (static_cast<int32_t>(blockIdx.x) >= blocks) return;
  int r = round0;
  int32_t m = n;
  CoreEnd end = kCoreHandOver;
  const int s = head ? 1 : 0;
  bool handed = head != nullptr;  // a stage has written colors
  if (head || n > kSmallMax) {
    end = core_stage<2, 2, kCoreThreads>(b, x.set[s], x.x[s], x.set[2], n, kSmallMax, r, round_cap, s_mask, sh.mid, &m,
                                         deadline);
    if (end == kCoreHandOver) {
      handed = true;
      core_hand_over(x.x[s].flag);
      if (blockIdx.x != 0) return;
      if (!core_take_over(x.x[s].flag, blocks, deadline, &s_ok)) end = kCoreFail;
    }
  } else if (blockIdx.x != 0) {
    return;
  }
  if (end == kCoreHandOver)
    end = core_small(b, x.set[head || n > kSmallMax ? 2 : 0], m, r, round_cap, sh.small);
  if (threadIdx.x != 0) return;
  if (end == kCoreFail || (end == kCoreSpread && handed)) {
    atomicOr(err, kErrTailBarrier);
  } else if (blockIdx.x == 0) {
    if (end == kCoreSpread) {
      atomicOr(err, kErrCoreWindow);
    } else {
      atomicMax(b.rounds_done, r - 1 + b.round_base);
      if (end == kCoreCapped) st_dev(left, 1);
    }
  }
}

// Marks the call's second launch as one that did not run.
__global__ void core_refused_kernel(int32_t* err) { atomicOr(err, kErrTailCheckin); }

namespace {

size_t round_up(size_t x) { return (x + 255) / 256 * 256; }

// Blocks of the first stage over n vertices, and the words of its exchange.
int32_t first_blocks(int32_t n) {
  return n <= kSmallMax ? 1 : n <= 16384 ? (n + 63) / 64 : (n + 95) / 96;
}
int32_t first_words(int32_t n) { return n <= kSmallMax ? 0 : (n <= 16384 ? 2 : 3) * first_blocks(n); }

// Lays the scratch out from base (may be null: sizes only).  The exchange
// words and the header are at its end, cleared as `words` 64-bit words.
size_t layout(char* base, int32_t n, CoreScratch* x, CoreHeader** head, uint64_t** clear, int32_t* words) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base + off;
    off += round_up(bytes);
    return p;
  };
  const int32_t size[kSets] = {n, n > kMidMax ? kMidMax : 0, n > kSmallMax ? kSmallMax : 0};
  for (int s = 0; s < kSets; ++s) {
    const size_t m = static_cast<size_t>(size[s]);
    x->set[s].v = reinterpret_cast<int32_t*>(take(4 * m));
    x->set[s].t = reinterpret_cast<int32_t*>(take(4 * m));
    x->set[s].fw = reinterpret_cast<uint64_t*>(take(8 * m));
    x->set[s].rows = reinterpret_cast<uint32_t*>(take(4 * m * static_cast<size_t>(row_words(size[s]))));
  }
  const size_t from = off;
  for (int s = 0; s < kSets - 1; ++s) {
    const size_t w = static_cast<size_t>(s == 0 ? first_words(n) : n > kMidMax ? kMidMax / 32 : 0);
    x->x[s].A = reinterpret_cast<uint64_t*>(take(8 * w * kCoreSlots));
    x->x[s].B = reinterpret_cast<uint64_t*>(take(8 * w * kCoreColorWords));
    x->x[s].ma = reinterpret_cast<uint64_t*>(take(8 * w));
    x->x[s].mb = reinterpret_cast<uint64_t*>(take(8 * w));
    x->x[s].flag = reinterpret_cast<uint64_t*>(take(8 * 256));
  }
  CoreHeader* h = reinterpret_cast<CoreHeader*>(take(sizeof(CoreHeader)));
  if (head) *head = h;
  if (clear) *clear = reinterpret_cast<uint64_t*>(base + from);
  if (words) *words = static_cast<int32_t>((off - from) / 8);
  return off;
}

}  // namespace

size_t core_scratch_bytes(int32_t n) {
  CoreScratch x;
  return layout(nullptr, n, &x, nullptr, nullptr, nullptr);
}

int core_blocks_resident() {
  static int cache = 0;
  if (cache == 0) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, core_wide_kernel<3, 12, 512>, 512, 0) != hipSuccess)
      cache = -1;
    else
      cache = per * cus > 0 ? per * cus : -1;
  }
  return cache;
}

bool launch_core(const KeySource& k, const IncBufs& b, const BinLayout& L, const int32_t cnt[kBins], int32_t n,
                 bool split, int round0, int round_cap, void* scratch, uint32_t* bar, int32_t* err, int32_t* left,
                 int32_t checkin_us, hipStream_t st) {
  if (n <= 0 || n > kCoreMax) return false;
  const uint64_t khz = wall_clock_khz();
  uint64_t deadline = khz * 1000ull * kTailBarrierSeconds;
  uint64_t checkin = checkin_us < 0 ? 0ull : khz * static_cast<uint64_t>(checkin_us) / 1000ull;
  CoreScratch x;
  CoreHeader* head = nullptr;
  uint64_t* clear = nullptr;
  int32_t words = 0;
  layout(static_cast<char*>(scratch), n, &x, &head, &clear, &words);
  CoreWorklist q;
  q.wl = b.wl_in;
  for (int i = 0; i < kBins; ++i) {
    q.off[i] = L.off[i];
    q.cnt[i] = cnt[i];
  }
  const dim3 rank_grid((n + kRankPer - 1) / kRankPer);
  if (k.prio && !k.rank)
    hipLaunchKernelGGL(core_rank_kernel<true>, rank_grid, dim3(kCoreThreads), 0, st, k, q, n, x.set[0].v, b.T, clear,
                       words);
  else
    hipLaunchKernelGGL(core_rank_kernel<false>, rank_grid, dim3(kCoreThreads), 0, st, k, q, n, x.set[0].v, b.T, clear,
                       words);
  hipLaunchKernelGGL(core_build_kernel, dim3((n + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), 0, st, b,
                     x.set[0], b.A_in, split ? 1 : 0, row_words(n), n);
  IncBufs bb = b;
  if (n > kMidMax) {
    void* args[] = {&bb, &x.set[0], &x.x[0], &x.set[1], &head, &n, &round0, &round_cap, &bar, &err, &left, &deadline,
                    &checkin};
    const bool two = n <= 16384;
    if (hipLaunchCooperativeKernel(two ? reinterpret_cast<const void*>(core_wide_kernel<2, 8, 1024>)
                                       : reinterpret_cast<const void*>(core_wide_kernel<3, 12, 512>),
                                   dim3(first_blocks(n)), dim3(two ? 1024 : 512), args, 0, st) != hipSuccess)
      return false;
  } else {
    head = nullptr;
  }
  void* args[] = {&bb, &x, &head, &n, &round0, &round_cap, &bar, &err, &left, &deadline, &checkin};
  const int grid = n > kMidMax ? kMidMax / 64 : n <= kSmallMax ? 1 : (n + 63) / 64;
  if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(core_kernel), dim3(grid), dim3(kCoreThreads), args, 0,
                                 st) != hipSuccess) {
    if (!head) return false;
    // the wide stage may have handed over, and its vertices cannot go on
    // elsewhere: as if this launch's check-in had failed
    (void)hipGetLastError();
    hipLaunchKernelGGL(core_refused_kernel, dim3(1), dim3(1), 0, st, err);
  }
  return true;
}

}  // namespace gcol
