// Runs the neighbourhood walks on the CPU on rows that end at entry INT_MAX,
// the largest a row offset can name.
#define EMU_MAIN
#include <hip/hip_runtime.h>

#include <sys/wait.h>
#include <unistd.h>

#include "round_steps.hpp"
#include "setup.hip"

#define blocks_for inc_blocks_for
#include "inc.hip"

using namespace gcol;

namespace {

// base[INT_MAX - n] .. base[INT_MAX - 1] are the n entries of a.
const int32_t* at_end(const std::vector<int32_t>& a) { return a.data() - (static_cast<int64_t>(INT_MAX) - static_cast<int64_t>(a.size())); }

// Vertex `len`'s first hop holds entries 0 .. len-1, the last ones of ci; entry u's
// second hop holds `second` entries from second * u on, the last ones of ci2.
struct Rows {
  std::vector<int32_t> ci, ci2, rp2;
  GraphView g{};
  int32_t v, beg;
  Rows(int mode, int32_t len, int32_t second) {
    for (int32_t u = 0; u < len; ++u) ci.push_back(u);
    for (int32_t x = 0; x < len * second; ++x) ci2.push_back(x);
    for (int32_t u = 0; u <= len; ++u) rp2.push_back(INT_MAX - (len - u) * second);
    v = std::max(len, len * second);
    beg = INT_MAX - len;
    g.n = g.limit = v + 1;
    g.ci = at_end(ci);
    g.ci2 = at_end(ci2);
    g.rp2 = rp2.data();
  }
};

template <int MODE, int G>
int64_t scan(Rows& r, int32_t* seen) {
  emu::launch(1, kBlock, [&] {
    if (static_cast<int>(threadIdx.x) >= G) return;
    scan_nbhd<MODE>(r.g, r.v, r.beg, INT_MAX, static_cast<int>(threadIdx.x), G,
                    [&](int32_t u) { return ++seen[u], 1; }, [](int32_t) { return false; });
  });
  return 0;
}

template <int MODE, int G>
int64_t walk(Rows& r, int32_t* seen) {
  std::vector<int32_t> row(2 * G);
  emu::launch(1, kWave, [&] {
    if (static_cast<int>(threadIdx.x) >= G) return;
    walk_two_hop<MODE, G>(r.g, r.v, r.beg, INT_MAX, row.data(), [&](const int32_t(&x)[4]) {
      for (int j = 0; j < 4; ++j)
        if (x[j] >= 0) ++seen[x[j]];
    });
  });
  return 0;
}

int64_t work(Rows& r, int G) {
  std::vector<int64_t> sum(G);
  emu::launch(1, kBlock, [&] {
    const int i = static_cast<int>(threadIdx.x);
    if (i < G) sum[i] = hop_work(r.g, r.beg, INT_MAX, i, G);
  });
  return std::accumulate(sum.begin(), sum.end(), int64_t{0});
}

// The set of v's two-hop members, as a list.
template <int MODE>
int64_t set(Rows& r, int32_t* seen) {
  const int32_t words = r.g.n / 32 + 1, v = r.v;
  std::vector<int32_t> rp(v + 2, r.beg), aoff(v + 2, 0), alen(v + 2), A(r.g.n);
  rp[v + 1] = INT_MAX;
  r.g.rp = rp.data();
  std::vector<uint32_t> bm(words);
  emu::launch(1, kSetThreads, [&] {
    inc_sets_kernel<MODE, kSetWordsSmall>(r.g, &v, 0, 1, bm.data(), words, aoff.data(), alen.data(), A.data());
  });
  for (int32_t i = 0; i < alen[v]; ++i) ++seen[A[i]];
  return 0;
}

template <int MODE>
int64_t one(int what, int G, Rows& r, int32_t* seen) {
  switch (what * 1000 + G) {
    case 1: return scan<MODE, 1>(r, seen);
    case 4: return scan<MODE, 4>(r, seen);
    case 64: return scan<MODE, 64>(r, seen);
    case 256: return scan<MODE, kBlock>(r, seen);
    case 1016: return walk<MODE, 16>(r, seen);
    case 1064: return walk<MODE, 64>(r, seen);
    case 3000: return set<MODE>(r, seen);
    default: return work(r, G);
  }
}

}  // namespace

// what: 0 scan_nbhd, 1 walk_two_hop, 2 hop_work, 3 inc_sets_kernel.  seen
// receives how often each id was visited; the result is hop_work's sum.  Runs in a
// child process; -1 if that died.
extern "C" int64_t walk_at_the_end(int what, int mode, int G, int32_t len, int32_t second, int32_t* seen) {
  Rows r(mode, len, second);
  const size_t bytes = sizeof(int64_t) + sizeof(int32_t) * (static_cast<size_t>(r.v) + 1);
  char* shared = static_cast<char*>(mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_SHARED | MAP_ANONYMOUS, -1, 0));
  int32_t* counts = reinterpret_cast<int32_t*>(shared + sizeof(int64_t));
  const pid_t pid = fork();
  if (pid == 0) {
    alarm(20);
    *reinterpret_cast<int64_t*>(shared) = mode == kD1   ? one<kD1>(what, G, r, counts)
                                          : mode == kD2 ? one<kD2>(what, G, r, counts)
                                                        : one<kPD2>(what, G, r, counts);
    _exit(0);
  }
  int status = 0;
  waitpid(pid, &status, 0);
  const int64_t result = status == 0 ? *reinterpret_cast<int64_t*>(shared) : -1;
  std::memcpy(seen, counts, bytes - sizeof(int64_t));
  munmap(shared, bytes);
  return result;
}
