// csrc/fold.h on the CPU.  Built as a shared library by tests/test_fold.py.
#include <cstring>

#include "wave_on_cpu.h"

namespace bpe {
struct OpAdd { static uint32_t apply(uint32_t a, uint32_t b) { return a + b; } };
static uint32_t wave_shift_up(uint32_t v, uint32_t identity) {
  const uint32_t before = __shfl_up(v, 1, 64);
  return threadIdx.x == 0 ? identity : before;
}
template <class Op>
static uint32_t wave_scan(uint32_t v, uint32_t) {
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t before = __shfl_up(v, d, 64);
    if ((int)threadIdx.x >= d) v = Op::apply(before, v);
  }
  return v;
}
}  // namespace bpe
static uint32_t __builtin_amdgcn_udot4(uint32_t a, uint32_t b, uint32_t c, bool) {
  for (int i = 0; i < 4; ++i) c += ((a >> 8 * i) & 255u) * ((b >> 8 * i) & 255u);
  return c;
}

#include "fold.h"

// text, marks (or null): padded by 16 bytes.  stretches: [64][5] x, out, q, first, end.  Returns their number, -1: not folded.
extern "C" int fold(const uint8_t* text, const uint8_t* marks, int n, int most, uint32_t* stretches, int* bytes) {
  static uint32_t lds[128];
  int result = 0;
  run_wave([&](int lane) {
    bpe::Fold f{};
    auto load = [&](int at) {
      uint4 v;
      std::memcpy(&v, text + at, 16);
      return v;
    };
    auto marked = [&](int at) {
      uint32_t m = 0;
      for (int j = 0; marks && j < 16; ++j) m |= (marks[at + j] ? 1u : 0u) << j;
      return m;
    };
    const bool folded = bpe::fold_text(n, most, lds, load, marked, f);
    uint32_t* const mine = stretches + 5 * lane;
    mine[0] = f.x; mine[1] = f.out; mine[2] = f.q; mine[3] = f.first; mine[4] = f.end;
    if (lane == 0) {
      result = folded ? f.stretches : -1;
      *bytes = f.bytes;
    }
  });
  return result;
}

extern "C" void block(uint64_t w, uint32_t size, uint32_t q, uint32_t least, uint32_t* at_and_bytes) {
  const bpe::FoldBlock b = bpe::fold_block(w, size, q, least);
  at_and_bytes[0] = b.at;
  at_and_bytes[1] = b.bytes;
}
