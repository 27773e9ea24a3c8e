// Waves on the CPU, for drivers that compile csrc headers without HIP: 64 lanes each, that exchange one value at every
// cross-lane operation.  A lane is a context of its own on one thread; it runs until it has to wait for the others.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <functional>
#include <memory>
#include <random>
#include <vector>

namespace {
struct Wave {
  int64_t slot[64];
  int arrived = 0;
  uint64_t steps = 0;                                  // that all lanes have made
};
struct Lane {
  ucontext_t context;
  std::unique_ptr<char[]> stack;
  Wave* wave;
  unsigned number;
  bool done = false;
};
Wave* my_wave;
Lane* my_lane;
struct { unsigned x; } threadIdx;                      // within the wave
ucontext_t scheduler;
const std::function<void()>* lane_work;

void let_others_run() { swapcontext(&my_lane->context, &scheduler); }
void wait_for_wave() {
  Wave& wave = *my_wave;
  const uint64_t step = wave.steps;
  if (++wave.arrived == 64) {
    wave.arrived = 0;
    ++wave.steps;
  }
  while (wave.steps == step) let_others_run();
}

int64_t from_lane(int64_t mine, int lane) {
  my_wave->slot[threadIdx.x] = mine;
  wait_for_wave();
  const int64_t got = my_wave->slot[lane];
  wait_for_wave();
  return got;
}
[[maybe_unused]] uint64_t __ballot(bool mine) {
  my_wave->slot[threadIdx.x] = mine;
  wait_for_wave();
  uint64_t mask = 0;
  for (int i = 0; i < 64; ++i) mask |= (uint64_t)my_wave->slot[i] << i;
  wait_for_wave();
  return mask;
}
template <class T>
T __shfl(T mine, int lane, int) { return (T)from_lane(mine, lane & 63); }
template <class T>
T __shfl_up(T mine, int d, int) { return (T)from_lane(mine, (int)threadIdx.x < d ? (int)threadIdx.x : (int)threadIdx.x - d); }
[[maybe_unused]] int __builtin_amdgcn_readlane(int mine, int lane) { return (int)from_lane(mine, lane); }
[[maybe_unused]] void __builtin_amdgcn_fence(int, const char*) {}
[[maybe_unused]] void __builtin_amdgcn_wave_barrier() { wait_for_wave(); }
[[maybe_unused]] uint32_t __builtin_amdgcn_alignbit(uint32_t high, uint32_t low, uint32_t shift) {
  return (uint32_t)(((uint64_t)high << 32 | low) >> (shift & 31));
}
struct uint4 { uint32_t x, y, z, w; };
[[maybe_unused]] uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
using std::max;
using std::min;

// work(wave, lane) in all lanes of n waves.  Lanes take their turns in order, those of several waves in a random one.
template <class Work>
void run_waves(int n, const Work& work) {
  constexpr size_t kStack = 256 << 10;
  static std::vector<Lane> lanes;
  std::vector<Wave> waves((size_t)n);
  lanes.resize(std::max(lanes.size(), (size_t)n * 64));
  const std::function<void()> body = [&] {
    work((int)(my_wave - waves.data()), (int)threadIdx.x);
    my_lane->done = true;
  };
  lane_work = &body;
  std::vector<Lane*> turns;
  for (int i = 0; i < n * 64; ++i) {
    Lane& lane = lanes[(size_t)i];
    if (!lane.stack) lane.stack = std::make_unique<char[]>(kStack);
    getcontext(&lane.context);
    lane.context.uc_stack.ss_sp = lane.stack.get();
    lane.context.uc_stack.ss_size = kStack;
    lane.context.uc_link = &scheduler;
    makecontext(&lane.context, [] { (*lane_work)(); }, 0);
    lane.wave = &waves[(size_t)(i / 64)];
    lane.number = (unsigned)i % 64;
    lane.done = false;
    turns.push_back(&lane);
  }
  std::mt19937 random(1);
  while (!turns.empty()) {
    if (n > 1) std::shuffle(turns.begin(), turns.end(), random);
    for (Lane* lane : turns) {
      my_lane = lane;
      my_wave = lane->wave;
      threadIdx.x = lane->number;
      swapcontext(&scheduler, &lane->context);
    }
    turns.erase(std::remove_if(turns.begin(), turns.end(), [](Lane* lane) { return lane->done; }), turns.end());
  }
}
template <class Work>
void run_wave(const Work& work) {
  run_waves(1, [&](int, int lane) { work(lane); });
}
}  // namespace

#define __device__
