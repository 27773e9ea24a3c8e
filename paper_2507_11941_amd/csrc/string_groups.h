// How a wave divides 64 neighbouring strings into groups: the work items of a batch of many short strings.  (No HIP
// header is included here, so that a host program that brings its own wave can compile this file.)
#pragma once
#include <stdint.h>

namespace bpe {

constexpr int kGroupBytes = 2048;                      // capacity of a work item ...
constexpr int kMemberBytes = 1024;                     // ... and of the strings or pieces in it
constexpr int kGroupLen = 0xFFF;                       // a group's ItemDesc::len: its length in bytes (kGroupLen: not
constexpr int kGroupShift = 12;                        //   encodable), its strings from bit kGroupShift on, and
constexpr int kGroupMask = 0x7F;                       //   kGroupApart once one of its strings had to be passed on: then
constexpr int kGroupApart = 1 << 30;                   //   each string's ids lie at its own place in the staging area
// The group that string s = tile + threadIdx.x heads; members = 0 if it heads none.  Whole waves take part.
struct StringGroup {
  int64_t begin;
  int members, len;
};
// Positions are compared relative to the wave's first byte, in 32 bits (in 64, 6,000 strings of up to 200 bytes took
// 48 us instead of 46).  Strings that end 2^28 bytes or more after it -- one among them is longer than the host said, and
// its own output is unspecified -- stay alone, with their own lengths, and so do those that are too long for a group
// themselves and those with offsets that decrease.
constexpr int64_t kGroupFar = (int64_t)1 << 28;
// The wave's n members lie one after the other, from `begin` to `end` each; those with `alone` set are groups of their
// own, wherever they lie, and with a negative room all are.
__device__ inline StringGroup group_members(int64_t begin, int64_t end, bool alone, int n, int room) {
  const int lane = threadIdx.x & 63;
  StringGroup g{begin, 0, kGroupLen};
  const uint64_t others = __ballot(lane < n && !alone);
  const int64_t base = __shfl(begin, others ? __builtin_ctzll(others) : 0, 64);
  alone = alone || begin < base || end < begin || end - base >= kGroupFar || end - begin > kMemberBytes;
  const uint64_t alone_lanes = __ballot(lane >= n || alone);
  const int from = alone ? 0 : (int)(begin - base), to = alone ? 0 : (int)(end - base);
  // Every lane looks for the end of a group that its string would head: the last string before the next one that is
  // alone (`to` does not decrease up to there) that still fits.  What is left to do one by one is a single hop a group.
  // (A walk that asks all lanes at every hop took 7 us for 64 groups of one string, in both kernels.)
  int last = lane;
  uint64_t heads = n >= 64 ? ~0ull : (1ull << n) - 1ull;
  if (room >= 0) {                                     // uniform
    const uint64_t alone_later = lane < 63 ? alone_lanes & (~0ull << (lane + 1)) : 0ull;
    const int limit = alone ? lane : alone_later ? __builtin_ctzll(alone_later) : 64;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) {
      const int its_end = __shfl(to, (last + step) & 63, 64);
      if (last + step < limit && its_end <= from + room) last += step;
    }
    uint64_t left = heads & ~alone_lanes;              // uniform: strings not alone that are in no group yet
    heads &= alone_lanes;
    while (left) {
      const int at = __builtin_ctzll(left), end_at = __builtin_amdgcn_readlane(last, at);
      heads |= 1ull << at;
      left &= end_at >= 63 ? 0ull : ~0ull << (end_at + 1);
    }
  }
  if ((heads >> lane) & 1ull) g.members = last + 1 - lane;
  const int64_t group_len = __shfl(end, max(lane + g.members - 1, 0), 64) - g.begin;
  if (g.members && group_len >= 0 && group_len <= (g.members > 1 ? kGroupBytes : kMemberBytes)) g.len = (int)group_len;
  return g;
}
__device__ inline StringGroup string_group(const int64_t* offsets, int64_t tile, int batch, int room) {
  const int lane = threadIdx.x & 63;
  const int64_t first = tile + (threadIdx.x & ~63u);   // the wave's first string ...
  const int n = (int)min((int64_t)batch - first, (int64_t)64);           // ... and how many it has (0 or less: none)
  if (n <= 0) return StringGroup{0, 0, kGroupLen};     // uniform
  int64_t begin = 0, end = 0;
  if (lane < n) {
    begin = offsets[first + lane];
    end = offsets[first + lane + 1];
  }
  return group_members(begin, end, false, n, room);
}

}  // namespace bpe
