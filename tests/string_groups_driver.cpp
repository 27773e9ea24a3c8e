// csrc/string_groups.h on the CPU.  Built as a shared library by tests/test_string_groups.py.
#include "wave_on_cpu.h"

#include "string_groups.h"

// members[s], len[s]: of the group that string s heads (0, unset: none); what one wave after the other finds.
extern "C" void string_groups(const int64_t* offsets, int batch, int room, int32_t* members, int32_t* len) {
  run_wave([=](int t) {
    for (int64_t tile = 0; tile < batch; tile += 64) {
      const bpe::StringGroup g = bpe::string_group(offsets, tile, batch, room);
      if (tile + t >= batch) continue;
      members[tile + t] = g.members;
      if (g.members) len[tile + t] = g.len;
    }
  });
}
