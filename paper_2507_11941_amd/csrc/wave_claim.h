// Numbers that waves take from a counter, one a wave and call.  (No HIP header is included here, so that a host program that
// brings its own waves can compile this file.)
#pragma once
#include <stdint.h>

namespace bpe {

// Counts one on and returns the number before, in all lanes; all lanes take part.  One lane alone goes to the counter, so that
// no other wave's numbers can come between.  What it adds is the same whichever lane it is: a number that depends on the lane (1 in one,
// 0 in the others) makes the compiler go over the 64 of them (some 640 scalar instructions, 1.3 us).  An increment that wraps
// (atomicInc) needs no such care, but where many waves go to one counter at a time it is served at half the rate: 600 items that do
// not fold were tried in 28 us instead of 16.
__device__ inline uint32_t wave_claim(uint32_t* counter) {
  // (The wave meets before and after the branch, so that the compiler joins it to no other lane's branch around the call: lanes
  // sent round a caller's loop on their own would miss the number.)
  __builtin_amdgcn_wave_barrier();
  uint32_t before = 0;
  if ((threadIdx.x & 63) == 0) before = atomicAdd(counter, 1u);
  __builtin_amdgcn_wave_barrier();
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
}

}  // namespace bpe
