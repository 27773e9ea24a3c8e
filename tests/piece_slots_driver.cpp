// csrc/piece_slots.h on the CPU.  Built as a shared library by tests/test_piece_slots.py.
#include "wave_on_cpu.h"

#include "piece_slots.h"

// What the kernels leave of every slot: as a list finds it (one wave, step after step, that starts to search anew at every
// `steps_each`-th) or, with steps_each 0, as a batch that is not listed does (a wave a slot).
extern "C" void piece_slots(const uint8_t* bytes, const int64_t* offsets, int batch, const uint8_t* cover, const uint32_t* cuts,
                            int piece_target, int max_string, uint32_t n_slots, uint32_t steps_each, int32_t* slot_string,
                            int64_t* piece_begin, int32_t* piece_len) {
  int32_t string_at[64];
  run_wave([&](int) {
    if (steps_each == 0) {
      for (uint32_t g = 0; g < n_slots; ++g)
        bpe::slot_piece(bytes, bpe::slot_string_of(offsets, batch, piece_target, g), cover, cuts, piece_target, max_string, g,
                        slot_string, piece_begin, piece_len);
      return;
    }
    int s0 = 0;
    for (uint32_t step = 0, g0 = 0; g0 < n_slots; ++step, g0 += bpe::kListSlots) {
      if (step % steps_each == 0)
        s0 = bpe::wave_last_string(batch, [&](int i) { return bpe::slot_base(offsets[i], i, piece_target) <= g0; });
      s0 = bpe::step_slots(bytes, offsets, batch, cover, cuts, piece_target, max_string, n_slots, g0, s0, string_at, slot_string,
                           piece_begin, piece_len).next_s0;
    }
  });
}

extern "C" bool small_batch(int64_t slots, int64_t resident, int64_t rest_grid) { return bpe::small_batch_fits(slots, resident, rest_grid); }
