// csrc/string_groups.h on the CPU: a wave is 64 threads that exchange one value each at every cross-lane operation.
// Built as a shared library by tests/test_string_groups.py.
#include <algorithm>
#include <barrier>
#include <cstdint>
#include <thread>
#include <vector>

namespace {
std::barrier<> wave_step(64);
int64_t wave_slot[64];
struct { unsigned x; } thread_local threadIdx;

int64_t from_lane(int64_t mine, int lane) {
  wave_slot[threadIdx.x] = mine;
  wave_step.arrive_and_wait();
  const int64_t got = wave_slot[lane];
  wave_step.arrive_and_wait();
  return got;
}
uint64_t __ballot(bool mine) {
  wave_slot[threadIdx.x] = mine;
  wave_step.arrive_and_wait();
  uint64_t mask = 0;
  for (int i = 0; i < 64; ++i) mask |= (uint64_t)wave_slot[i] << i;
  wave_step.arrive_and_wait();
  return mask;
}
template <class T>
T __shfl(T mine, int lane, int) { return (T)from_lane(mine, lane); }
int __builtin_amdgcn_readlane(int mine, int lane) { return (int)from_lane(mine, lane); }
using std::max;
using std::min;
}  // namespace

#define __device__
#include "string_groups.h"

// members[s], len[s]: of the group that string s heads (0, unset: none); what one wave after the other finds.
extern "C" void string_groups(const int64_t* offsets, int batch, int room, int32_t* members, int32_t* len) {
  std::vector<std::thread> lanes;
  for (unsigned t = 0; t < 64; ++t)
    lanes.emplace_back([=] {
      threadIdx.x = t;
      for (int64_t tile = 0; tile < batch; tile += 64) {
        const bpe::StringGroup g = bpe::string_group(offsets, tile, batch, room);
        if (tile + t >= batch) continue;
        members[tile + t] = g.members;
        if (g.members) len[tile + t] = g.len;
      }
    });
  for (std::thread& t : lanes) t.join();
}
