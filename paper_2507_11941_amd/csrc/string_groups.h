// How a wave divides 64 neighbouring strings into groups: the work items of a batch of many short strings.  (No HIP
// header is included here, so that a host program that brings its own wave can compile this file.)
#pragma once
#include <stdint.h>

namespace bpe {

constexpr int kGroupBytes = 1024;                      // capacity of a work item
constexpr int kGroupLen = 0xFFF;                       // a group's ItemDesc::len: its length in bytes (kGroupLen: not
constexpr int kGroupShift = 12;                        //   encodable), its strings from bit kGroupShift on, and
constexpr int kGroupMask = 0x7F;                       //   kGroupApart once one of its strings had to be passed on: then
constexpr int kGroupApart = 1 << 30;                   //   each string's ids lie at its own place in the staging area
// The group that string s = tile + threadIdx.x heads; members = 0 if it heads none.  Whole waves take part.
struct StringGroup {
  int64_t begin;
  int members, len;
};
// The walk compares positions relative to the wave's first byte in 32 bits (in 64, 6,000 strings of up to 200 bytes took
// 48 us instead of 46).  Strings that end 2^28 bytes or more after it -- one among them is longer than the host said, and
// its own output is unspecified -- stay alone, with their own lengths, and so do those with offsets that decrease.
constexpr int64_t kGroupFar = (int64_t)1 << 28;
__device__ inline StringGroup string_group(const int64_t* offsets, int64_t tile, int batch, int room) {
  const int lane = threadIdx.x & 63;
  const int64_t first = tile + (threadIdx.x & ~63u);   // the wave's first string ...
  const int n = (int)min((int64_t)batch - first, (int64_t)64);           // ... and how many it has (0 or less: none)
  StringGroup g{0, 0, kGroupLen};
  if (n <= 0) return g;                                // uniform
  const int64_t base = offsets[first];
  int64_t end = 0;
  if (lane < n) {
    g.begin = offsets[first + lane];
    end = offsets[first + lane + 1];
  }
  const bool alone = g.begin < base || end < g.begin || end - base >= kGroupFar;
  const uint64_t alone_lanes = __ballot(lane >= n || alone);
  const int from = alone ? 0 : (int)(g.begin - base), to = alone ? 0 : (int)(end - base);
  uint64_t heads = 0;
  for (int at = 0; at < n;) {                          // uniform; `at` grows every round
    heads |= 1ull << at;
    const uint64_t later = at < 63 ? ~0ull << (at + 1) : 0ull;
    uint64_t stop = (__ballot(to > __builtin_amdgcn_readlane(from, at) + room) | alone_lanes) & later;
    if ((alone_lanes >> at) & 1ull) stop = later;
    at = stop ? __builtin_ctzll(stop) : 64;
  }
  if ((heads >> lane) & 1ull) {
    const uint64_t later = lane < 63 ? heads & (~0ull << (lane + 1)) : 0ull;
    g.members = (later ? __builtin_ctzll(later) : n) - lane;
  }
  const int64_t group_len = __shfl(end, max(lane + g.members - 1, 0), 64) - g.begin;
  if (g.members && group_len >= 0 && group_len <= kGroupBytes) g.len = (int)group_len;
  return g;
}

}  // namespace bpe
