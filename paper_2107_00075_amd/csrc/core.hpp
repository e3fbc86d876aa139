// Interface of the core kernels (core.hip): the remaining rounds of a call
// whose worklist has shrunk to a few thousand vertices.
#pragma once

#include "inc.hpp"

namespace gcol {

constexpr int kCoreSlots = 32;          // color classes in flight: the spread of the tentative colors
constexpr int32_t kCoreMax = 24576;     // vertices: 96 per workgroup, one workgroup on each of 256 CUs
constexpr int32_t kCoreMid = 4096;    // above: two cooperative launches
constexpr int32_t kCoreSmall = 1024;  // up to here: one workgroup, which takes any spread of the colors
constexpr int32_t kErrCoreWindow = 0x400;  // error bit: the tentative colors spread over more than kCoreSlots colors
constexpr int32_t kErrCoreHanded = 0x800;  // (no error) the wide stage has written colors and handed over

// Vertices a launch of `blocks` workgroups can take.
inline int32_t core_capacity(int blocks) {
  return blocks >= 256 ? kCoreMax : blocks >= 64 ? 64 * blocks : blocks > 0 ? kCoreSmall : 0;
}

// Bytes of the scratch one launch over n vertices needs: the vertices in key
// order, their rows of adjacency bits and the exchange words.
size_t core_scratch_bytes(int32_t n);

// Workgroups of the core kernel that fit on the device at once (-1: unknown).
int core_blocks_resident();

// Colors the n vertices of the worklist b.wl_in (bin regions L.off, cnt[]
// entries each; round round0's worklist) in one or two cooperative launches
// (after two launches that set them up), unless they are refused (false).  *err receives
// kErrTailCheckin (not all workgroups were resident), kErrCoreWindow or
// kErrTailBarrier (a wait gave up); with the first two, unless kErrCoreHanded
// is there too, nothing that the rounds read has been written.  split: the lists are split by key (higher
// part in front, lower part at the back), else they are one part of length
// alen_in.
bool launch_core(const KeySource& k, const IncBufs& b, const BinLayout& L, const int32_t cnt[kBins], int32_t n,
                 bool split, int round0, int round_cap, void* scratch, uint32_t* bar, int32_t* err, int32_t* left,
                 int32_t checkin_us, hipStream_t st);
inline int core_launches(int32_t n) { return n > kCoreMid ? 4 : 3; }

}  // namespace gcol
