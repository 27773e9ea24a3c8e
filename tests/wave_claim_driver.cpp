// csrc/wave_claim.h on the CPU: two waves that claim from one counter.  Built as a shared library by tests/test_wave_claim.py.
#include "wave_on_cpu.h"

// As the memory serves them: one lane's after the other, in any order among the lanes of both waves.
static uint32_t atomicAdd(uint32_t* at, uint32_t each) {
  let_others_run();
  const uint32_t before = *at;
  *at += each;
  return before;
}
static int __builtin_amdgcn_readfirstlane(int mine) { return __builtin_amdgcn_readlane(mine, 0); }

#include "wave_claim.h"

// taken: [waves][64][times], what each lane got.  Returns the counter's last value.
extern "C" uint32_t claims(int waves, int times, uint32_t* taken) {
  uint32_t counter = 0;
  run_waves(waves, [&](int wave, int lane) {
    for (int i = 0; i < times; ++i) taken[(wave * 64 + lane) * times + i] = bpe::wave_claim(&counter);
  });
  return counter;
}
