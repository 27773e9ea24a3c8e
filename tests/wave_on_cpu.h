// Waves on the CPU: 64 threads each that exchange one value at every cross-lane operation, for drivers that compile csrc
// headers without HIP.
#pragma once
#include <algorithm>
#include <barrier>
#include <cstdint>
#include <thread>
#include <vector>

namespace {
struct Wave {
  std::barrier<> step{64};
  int64_t slot[64];
};
thread_local Wave* my_wave;
struct { unsigned x; } thread_local threadIdx;           // within the wave

int64_t from_lane(int64_t mine, int lane) {
  my_wave->slot[threadIdx.x] = mine;
  my_wave->step.arrive_and_wait();
  const int64_t got = my_wave->slot[lane];
  my_wave->step.arrive_and_wait();
  return got;
}
[[maybe_unused]] uint64_t __ballot(bool mine) {
  my_wave->slot[threadIdx.x] = mine;
  my_wave->step.arrive_and_wait();
  uint64_t mask = 0;
  for (int i = 0; i < 64; ++i) mask |= (uint64_t)my_wave->slot[i] << i;
  my_wave->step.arrive_and_wait();
  return mask;
}
template <class T>
T __shfl(T mine, int lane, int) { return (T)from_lane(mine, lane); }
template <class T>
T __shfl_up(T mine, int d, int) { return (T)from_lane(mine, (int)threadIdx.x < d ? (int)threadIdx.x : (int)threadIdx.x - d); }
[[maybe_unused]] int __builtin_amdgcn_readlane(int mine, int lane) { return (int)from_lane(mine, lane); }
[[maybe_unused]] void __builtin_amdgcn_fence(int, const char*) {}
[[maybe_unused]] void __builtin_amdgcn_wave_barrier() { my_wave->step.arrive_and_wait(); }
[[maybe_unused]] uint32_t __builtin_amdgcn_alignbit(uint32_t high, uint32_t low, uint32_t shift) {
  return (uint32_t)(((uint64_t)high << 32 | low) >> (shift & 31));
}
struct uint4 { uint32_t x, y, z, w; };
[[maybe_unused]] uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
using std::max;
using std::min;

template <class Work>
void run_waves(int n, const Work& work) {
  std::vector<Wave> waves((size_t)n);               // (constructed in place: a barrier does not move)
  std::vector<std::thread> lanes;
  for (int w = 0; w < n; ++w)
    for (unsigned t = 0; t < 64; ++t)
      lanes.emplace_back([&, w, t] {
        my_wave = &waves[(size_t)w];
        threadIdx.x = t;
        work(w, (int)t);
      });
  for (std::thread& t : lanes) t.join();
}
template <class Work>
void run_wave(const Work& work) {
  run_waves(1, [&](int, int lane) { work(lane); });
}
}  // namespace

#define __device__
