// csrc/fold.h on the CPU.  Built by tests/test_fold.py as a shared library, and as a program with the sanitizers in it.
#include <cstdio>
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
static uint32_t lane_read(uint32_t v, int lane) { return __shfl(v, lane, 64); }
}  // namespace bpe
#define __forceinline__ inline
static void atomicOr(uint32_t* at, uint32_t bits) { *at |= bits; }
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

// The ids of a text by way of its folded one: sizes, ids: the `tokens` tokens of what stays of it.  Returns how many there are, -1: it
// does not fold or a stretch has no block.  Everything is as large as it has to be, for the sanitizers' sake; out: of `room` ids.
static int emit(const uint8_t* text, int n, const int32_t* sizes, const int32_t* ids, int tokens, int32_t* out, int room) {
  std::vector<uint32_t> T(64 * 16, 0xABCDEFu), lds(bpe::kFoldWords), search(128);
  int result = -1;
  run_wave([&](int lane) {
    bpe::Fold f{};
    auto load = [&](int at) {
      uint8_t sixteen[16] = {};
      std::memcpy(sixteen, text + at, (size_t)min(n - at, 16));
      uint4 v;
      std::memcpy(&v, sixteen, 16);
      return v;
    };
    if (!bpe::fold_text(n, bpe::kFoldBytes, search.data(), load, [](int) { return 0u; }, f) || f.stretches == 0) return;
    const int d = (f.bytes + 63) / 64;
    uint32_t live = 0, before = 0;
    int at = 0;
    for (int i = 0; i < tokens; at += sizes[i++]) {
      if (at / d < lane) ++before;
      if (at / d != lane) continue;
      live |= 1u << (at % d);
      T[(size_t)(64 * (at % d) + lane)] = 0x5A000000u | (uint32_t)ids[i];
    }
    bpe::wave_order();
    uint32_t total = (uint32_t)tokens;
    const bool done = bpe::emit_folded(f, live, T.data(), lds.data(), d, before, out, &total);
    if (lane == 63 && done) result = (int)total <= room ? (int)total : -2;
  });
  return result;
}

#ifdef FOLD_PROGRAM
// Standard input: n, tokens, room; the text, the tokens' sizes and ids.  Output: the number of ids, and they.
int main() {
  int32_t head[3];
  while (std::fread(head, sizeof head, 1, stdin) == 1) {
    std::vector<uint8_t> text((size_t)head[0]);
    std::vector<int32_t> sizes((size_t)head[1]), ids((size_t)head[1]), out((size_t)head[2], -1);
    if (std::fread(text.data(), 1, text.size(), stdin) != text.size() || std::fread(sizes.data(), 4, sizes.size(), stdin) != sizes.size() ||
        std::fread(ids.data(), 4, ids.size(), stdin) != ids.size())
      return 1;
    const int32_t k = emit(text.data(), head[0], sizes.data(), ids.data(), head[1], out.data(), head[2]);
    std::fwrite(&k, 4, 1, stdout);
    if (k > 0) std::fwrite(out.data(), 4, (size_t)k, stdout);
  }
  return 0;
}
#endif
