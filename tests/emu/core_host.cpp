// Runs core.hip's launch_core on the CPU: the rounds of a distance-1 graph
// from a start state, as the incremental engine hands it over.
#define EMU_MAIN
#include <hip/hip_runtime.h>

#include "core.hip"

namespace gcol {
uint64_t wall_clock_khz() { return 100000; }
}  // namespace gcol

using namespace gcol;

// init: 0 or the color of a committed vertex.  prio (nullable): explicit keys.
// colors, rounds, left (1: stopped at max_rounds): results.  Returns launch_core's error
// bits, or -1 if it refused.
extern "C" int core_run(int32_t n, const int32_t* rp, const int32_t* ci, uint32_t seed, const uint32_t* prio,
                        const int32_t* init, int32_t max_rounds, uint64_t order, int32_t* colors, int32_t* rounds,
                        int64_t* visits, int32_t* left) {
  emu::add_kernel(core_wide_kernel<2, 8, 1024>);
  emu::add_kernel(core_wide_kernel<3, 12, 512>);
  emu::add_kernel(core_kernel);
  emu::seed = order;
  std::vector<int32_t> T(n), work(n), len(n), wl, fw_off(n + 1);
  std::vector<uint32_t> done(n / 32 + 1);
  for (int32_t v = 0; v < n; ++v) {
    const int32_t d = rp[v + 1] - rp[v];
    colors[v] = T[v] = init ? init[v] : 0;
    work[v] = len[v] = d;
    fw_off[v + 1] = fw_off[v] + std::min(d, n) / 32;
    if (colors[v]) done[v >> 5] |= 1u << (v & 31);
    else wl.push_back(v);
  }
  std::vector<uint32_t> F(n + fw_off[n] + 1);
  for (int32_t v = 0; v < n; ++v) {
    for (int32_t e = rp[v]; e < rp[v + 1]; ++e) {
      const int32_t c = colors[ci[e]];
      if (c == 0) continue;
      const int32_t w = (c - 1) / 32;
      if (w == 0) F[v] |= 1u << (c - 1);
      else if (w <= fw_off[v + 1] - fw_off[v]) F[n + fw_off[v] + w - 1] |= 1u << ((c - 1) % 32);
    }
  }
  int32_t maxc = 0, light = 0, tile[2] = {}, err = 0;
  *rounds = *left = 0;
  std::vector<unsigned long long> acc(kAccSlots * kAccStride);
  std::vector<uint32_t> bar(kBarWords);
  IncBufs b{};
  b.C = colors;
  b.T = T.data();
  b.work = work.data();
  b.wl_in = wl.data();
  b.tile_ctr = tile;
  b.light_ctr = &light;
  b.aoff = rp;
  b.A_in = ci;
  b.alen_in = len.data();
  b.done = done.data();
  b.fw_off = fw_off.data();
  b.F = F.data();
  b.Fx = F.data() + n;
  b.maxc = &maxc;
  b.acc = acc.data();
  b.rounds_done = rounds;
  KeySource k{prio, nullptr, hash_seed(seed), nullptr};
  BinLayout L{};
  const int32_t left0 = static_cast<int32_t>(wl.size());
  const int32_t cnt[kBins] = {left0};
  std::vector<uint64_t> scratch(core_scratch_bytes(left0) / 8 + 1, 0xA5A5A5A5A5A5A5A5ull);
  if (!launch_core(k, b, L, cnt, left0, false, 1, max_rounds > 0 ? max_rounds : INT_MAX, scratch.data(), bar.data(),
                   &err, left, 60000000, nullptr))
    return -1;
  *visits = 0;
  for (int s = 0; s < kAccSlots; ++s) *visits += static_cast<int64_t>(acc[s * kAccStride]);
  return err;
}

// The second launch of a call of two, after a first one that ended with the
// error bits err and whose workgroup 0 handed n isolated vertices over.
// colors receives what it wrote.  Returns the error bits afterwards.
extern "C" int core_second_launch(int32_t n, int32_t err, int32_t* colors) {
  emu::seed = 1;
  const int32_t all = kMidMax + 64;  // vertices of the first launch
  std::vector<uint64_t> scratch(core_scratch_bytes(all) / 8 + 1);
  CoreScratch x;
  CoreHeader* head;
  uint64_t* clear;
  int32_t words;
  layout(reinterpret_cast<char*>(scratch.data()), all, &x, &head, &clear, &words);
  for (int32_t v = 0; v < n; ++v) {
    x.set[1].v[v] = v;
    x.set[1].t[v] = 1;
  }
  head->handed = 1;
  head->left = n;
  head->round = 5;
  std::vector<int32_t> work(n), fw_off(n + 1);
  std::vector<uint32_t> F(n + 1), bar(kBarWords);
  std::vector<unsigned long long> acc(kAccSlots * kAccStride);
  int32_t maxc = 0, rounds = 0, left = 0;
  IncBufs b{};
  b.C = colors;
  b.work = work.data();
  b.fw_off = fw_off.data();
  b.F = F.data();
  b.Fx = F.data() + n;
  b.maxc = &maxc;
  b.acc = acc.data();
  b.rounds_done = &rounds;
  emu::launch(dim3(kMidMax / 64), dim3(kCoreThreads),
              [&] { core_kernel(b, x, head, all, 1, INT_MAX, bar.data(), &err, &left, 3000000000u, 6000000000u); }, true);
  return err;
}
