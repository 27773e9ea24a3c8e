// Folding: text that repeats itself is encoded with most of its repetitions left out, and their tokens are put back in.
// (No HIP header is included here, so that a host program that brings its own wave can compile this file.)
//
// Why the result is Algorithm 1's.  A sequence of tokens is Algorithm 1's encoding of its bytes if and only if that is so for
// every two neighbours in it: the first merge that joined bytes across a boundary of the sequence would, with everything
// around taken away, be made of those two tokens' bytes as well, since until then nothing has crossed a boundary and what
// happens inside the two tokens does not depend on what lies beyond them; the other way round, where no boundary is crossed
// in the whole text, none is in a part of it.  So if the encoding of a text holds a block of tokens twice in a row, more
// copies of that block put in behind the second one make no new neighbours, and the longer sequence is the encoding of the
// longer text.
//
// A stretch is text that equals itself `q` bytes earlier, q up to kFoldPeriods (blank or padded records, separator lines,
// repeated markup).  Of a long one all but its first q + 23 bytes and a remainder is left out, in whole units of fold_unit(q)
// bytes.  The rest is encoded; in the stretch's tokens a block of B bytes is looked for that is there twice in a row, with B
// a multiple of q that divides what was left out (a token's bytes say which token it is, so that the places where tokens
// start tell all); and (what was left out) / B copies of it are written.  If a stretch has no such block, which a table
// with tokens longer than the part that stays can bring about, the text is encoded as it is.
#pragma once
#include <stdint.h>

#include "piece_slots.h"

namespace bpe {

// Two words of history: a lane's sixteen bytes are compared with those up to eight earlier by shifts of six words, two periods to a
// result word (fold_equal), and each further period would cost every text that comes here, and two more words to hand on.  Longer
// motifs are encoded as they are: 600 strings of 16,000 bytes take 81 us with a period of 8, 197 to 208 with 9, 12 or 16.
constexpr int kFoldPeriods = 8;
constexpr int kFoldHistory = 24;                       // repeating bytes from which on the next ones may be left out
constexpr int kFoldStretches = 64;                     // of a text: a lane each
constexpr int kFoldBytes = 1024;                       // most that may stay of a text: sixteen bytes a lane
// A lane's sixteen bytes of a folded text and their two neighbours are to hold one place at most where bytes are left out.
constexpr uint32_t kFoldApart = 18;
// A text of fewer bytes is taken as it is, two a lane at most: looking for stretches takes a wave 2 us, which rows of words with
// a long one among them pay for nothing (20,011 of up to 60 bytes, one in twenty with such a word: 64.9 us with 96, 63.0 so).
constexpr int kFoldLeast = 128;

// Bytes left out of a stretch are a multiple of this: q by a power of two, at most 16.
__device__ inline uint32_t fold_unit(uint32_t q) { return q <= 2 ? 8u : 2u * q; }

// A wave's folded text; lane j has stretch j.
struct Fold {
  int stretches;                                       // (uniform) 0: nothing is left out
  int bytes;                                           // (uniform) that stay
  uint32_t x, out;                                     // place in the folded text where bytes are left out, and how many
  uint32_t q, first, end;                              // period; the stretch's first byte in the folded text, and its end
};

// Which of a lane's sixteen bytes, w[2 ... 5], equal the one q bytes earlier, bit j: byte j, for q up to 4, and for q + 4 in the
// high half; w[0] and w[1] are the eight bytes before.
__device__ inline uint32_t fold_equal(const uint32_t (&w)[6], uint32_t q) {
  uint32_t differ[2] = {0, 0};
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    uint32_t low = 0, high = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // (by four: the low word itself)
      const uint32_t earlier = __builtin_amdgcn_alignbit(w[k + 2 - half], w[k + 1 - half], (32u - 8u * q) & 31u);
      const uint32_t d = w[k + 2] ^ earlier;
      const uint32_t nonzero = ((((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | d) >> 7) & 0x01010101u;
      uint32_t& to = k < 2 ? low : high;
      to = __builtin_amdgcn_udot4(nonzero, k & 1 ? 0x80402010u : 0x08040201u, to, false);
    }
    differ[half] = low | high << 8;
  }
  return ~(differ[0] | differ[1] << 16);
}

// Whether some of a lane's sixteen bytes may be repeating ones: of a run of 24 bytes that equal those q earlier, q up to 8, eight
// in an aligned place at least equal those 5, 6, 7 or 8 earlier (a multiple of q; up to four of the 24 are lost to it).
__device__ inline bool fold_possible(const uint32_t (&w)[6]) {
  uint32_t least = ~0u;
#pragma unroll
  for (uint32_t q = 5; q <= 8; ++q) {
    uint32_t differ[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) differ[k] = w[k + 2] ^ __builtin_amdgcn_alignbit(w[k + 1], w[k], (32u - 8u * q) & 31u);
    least = min(least, min(differ[0] | differ[1], differ[2] | differ[3]));
  }
  return least == 0;
}

// Finds the stretches of a text of n bytes, a wave's work.  load(at): the sixteen bytes from `at` on, at < n, for all lanes
// at once; marked(at): a bit for each of those bytes that is part of a special token, which no stretch holds.  lds: 128 words.
// Returns false where more than `most` bytes or kFoldStretches stretches stay.
//
// A wave looks at 1 KiB at a time.  Byte i may be left out with period q if the 24 bytes up to it equal those q earlier; the
// smallest such q is taken (of a stretch whose least period is g, the multiples of g begin later and end with it, and no
// other period holds for as long).  A lane's sixteen bytes have at most one run of such bytes: two stretches overlap by less
// than their periods, so that after the end of one, 16 bytes at least lie before the first byte of the next that may go (and
// places in the folded text where bytes are left out lie 16 apart; should they be nearer than kFoldApart, which takes two
// stretches that share seven bytes, the text is not folded).
// Most text of up to 1 KiB that comes here does not repeat itself, and is first looked at roughly (fold_possible): 20,000 strings of
// 300 bytes without a cut 264 -> 255 us.  (Of longer text two rows tell; a rough look at those gained nothing.)
// Where a whole KiB continues a stretch, only its own period is asked, four such rows in flight: 64 KiB of one byte takes
// 64 rows, and 256 such strings a wave each.
template <class Load, class Marked>
__device__ inline bool fold_text(int n, int most, uint32_t* lds, const Load& load, const Marked& marked, Fold& f) {
  const int lane = (int)threadIdx.x & 63;
  uint32_t* const starts = lds;                        // first byte that may be left out | period << 20
  uint32_t* const ends = lds + 64;
  uint32_t before_z = 0, before_w = 0;                 // the eight bytes before the row (uniform)
  uint32_t last1[4] = {0, 0, 0, 0}, last2[4] = {0, 0, 0, 0};   // of the lane before the row, and the one before that (uniform)
  uint32_t marked_before = 0;
  int count = 0, stay = 0;                             // stretches; bytes that are sure to stay (uniform)
  uint32_t open_q = 0;                                 // period of the stretch that the row's end lies in, 0: none (uniform)
  uint4 only = make_uint4(0, 0, 0, 0);                 // the row of a text that has just one
  if (n <= 1024) {                                     // uniform
    if (16 * lane < n) only = load(16 * lane);
    const uint32_t words[6] = {wave_shift_up(only.z, 0u), wave_shift_up(only.w, 0u), only.x, only.y, only.z, only.w};
    if (!__ballot(fold_possible(words) && 16 * lane < n)) {                // uniform
      f.stretches = 0;
      f.bytes = n;
      return n <= most;
    }
  }
  // (the row that begins at n, if n is a whole number of rows, ends a stretch that reaches it)
  for (int row = 0; row <= n;) {                       // uniform
    if (open_q != 0) {
      // ---- rows that continue the stretch from end to end ----
      for (;;) {                                       // uniform
        const int rows = min((n - row) >> 10, 4);
        if (rows <= 0) break;
        uint4 v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r < rows) v[r] = load(row + 1024 * r + 16 * lane);
        int whole = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (r < rows && whole == r) {                // uniform
            const uint32_t z = wave_shift_up(v[r].z, before_z), w = wave_shift_up(v[r].w, before_w);
            const uint32_t words[6] = {z, w, v[r].x, v[r].y, v[r].z, v[r].w};
            const uint32_t shift = (32u - 8u * open_q) & 31u;                    // (period 4 and 8: a whole word)
            uint32_t d = marked(row + 1024 * r + 16 * lane);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const uint32_t high = open_q > 4 ? words[k + 1] : words[k + 2], low = open_q > 4 ? words[k] : words[k + 1];
              d |= words[k + 2] ^ __builtin_amdgcn_alignbit(high, low, shift);
            }
            if (!__ballot(d != 0)) {
              ++whole;
              before_z = (uint32_t)__builtin_amdgcn_readlane((int)v[r].z, 63);
              before_w = (uint32_t)__builtin_amdgcn_readlane((int)v[r].w, 63);
            }
          }
        }
        row += 1024 * whole;
        if (whole > 0) {                               // what is known of the lanes before the next row
          const uint32_t full = open_q > 4 ? 0xFFFF0000u : 0xFFFFu;
          for (int k = 0; k < 4; ++k) last1[k] = last2[k] = k == (int)((open_q - 1u) & 3u) ? full : 0u;
          marked_before = 0;
        }
        if (whole < rows) break;
      }
    }
    // ---- a row of its own ----
    const int at = row + 16 * lane;
    uint4 v = make_uint4(0, 0, 0, 0);
    uint32_t mark = 0;
    if (at < n) {
      v = n <= 1024 ? only : load(at);                 // (uniform)
      mark = marked(at);
    }
    const uint32_t z = wave_shift_up(v.z, before_z), w = wave_shift_up(v.w, before_w);
    const uint32_t words[6] = {z, w, v.x, v.y, v.z, v.w};
    const int here = n - at;                           // bytes of the text from my first one on
    uint32_t within = here >= 16 ? 0xFFFFu : here > 0 ? (1u << here) - 1u : 0u;
    {                                                  // neither a mark nor the eight bytes after one
      const uint32_t m = wave_shift_up(mark, marked_before) | mark << 16;
      uint32_t near = m | m << 1;
      near |= near << 2;
      near |= near << 4;
      near |= m << 8;
      within &= ~(near >> 16);
      marked_before = (uint32_t)__builtin_amdgcn_readlane((int)mark, 63);
    }
    if (row == 0 && lane == 0) within &= ~((1u << kFoldPeriods) - 1u);           // (nothing lies before the text)
    uint32_t same[4], one[4], two[4];                  // of my bytes, and those of the two lanes before me; two periods each
    bool some = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      same[k] = fold_equal(words, (uint32_t)k + 1u) & (within | within << 16);
      one[k] = wave_shift_up(same[k], last1[k]);
      two[k] = wave_shift_up(one[k], last2[k]);
      last1[k] = (uint32_t)__builtin_amdgcn_readlane((int)same[k], 63);
      last2[k] = (uint32_t)__builtin_amdgcn_readlane((int)same[k], 62);
      some = some || (one[k] & 0xFF00u) == 0xFF00u || one[k] >> 24 == 0xFFu;
    }
    before_z = (uint32_t)__builtin_amdgcn_readlane((int)v.z, 63);
    before_w = (uint32_t)__builtin_amdgcn_readlane((int)v.w, 63);
    uint32_t q = 0, lo = 0, hi = 0;                    // my bytes lo ... hi - 1 may be left out, with period q (0: none may)
    bool runs_on = false;                              // ... and so may the byte before mine
    if (__ballot(some)) {                              // uniform
#pragma unroll
      for (int c = kFoldPeriods; c >= 1; --c) {        // the smallest one is the last to be asked
        const int k = (c - 1) & 3, shift = c > 4 ? 16 : 0;
        const uint32_t mine = (same[k] >> shift) & 0xFFFFu;
        const uint32_t earlier = shift ? (one[k] & 0xFFFF0000u) | two[k] >> 16 : one[k] << 16 | (two[k] & 0xFFFFu);
        const uint32_t run = earlier == ~0u ? 32u : (uint32_t)__builtin_clz(~earlier);      // repeating bytes before mine
        const bool on = run >= (uint32_t)kFoldHistory;
        const uint32_t from = on ? 0u : (uint32_t)kFoldHistory - 1u - run;
        const uint32_t to = (uint32_t)__builtin_ctz(~mine);
        if (on || from < to) {
          q = (uint32_t)c;
          lo = from;
          hi = to;
          runs_on = on;
        }
      }
    }
    const bool begins = q != 0 && !runs_on, stops = q != 0 && hi < 16u;
    const uint64_t all_begin = __ballot(begins);
    const uint64_t below = lane == 63 ? ~0ull >> 1 : (1ull << lane) - 1ull;
    const int mine = count + (int)__builtin_popcountll(all_begin & below) + (begins ? 1 : 0) - 1;
    count += (int)__builtin_popcountll(all_begin);
    if (count > kFoldStretches) return false;          // uniform
    if (begins) starts[mine] = (uint32_t)at + lo | q << 20;
    if (stops) ends[mine] = (uint32_t)at + hi;
    stay += 16 * (int)__builtin_popcountll(__ballot(q == 0 && here >= 16));
    if (stay > most) return false;                     // uniform
    const uint32_t end_q = q != 0 && hi == 16u ? q : 0u;
    open_q = (uint32_t)__builtin_amdgcn_readlane((int)end_q, 63);
    row += 1024;
  }
  wave_order();
  f.stretches = count;
  const uint32_t start = lane < count ? starts[lane] : 0u, end = lane < count ? ends[lane] : 0u;
  wave_order();
  const uint32_t at = start & 0xFFFFFu, unit = fold_unit(max(start >> 20, 1u));
  f.q = start >> 20;
  f.out = lane < count ? (end - at) / unit * unit : 0u;
  const uint32_t upto = wave_scan<OpAdd>(f.out, 0u);
  f.x = at - (upto - f.out);
  f.first = f.x - (uint32_t)(kFoldHistory - 1) - f.q;
  f.end = f.x + (end - at) - f.out;
  f.bytes = n - (int)(uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  if (f.bytes == n) f.stretches = 0;
  const uint32_t x_before = wave_shift_up(f.x, 0u);
  return f.bytes <= most && !__ballot(lane > 0 && lane < count && f.x - x_before < kFoldApart);
}

// A block that a stretch's tokens hold twice in a row: bit i of w says that a token starts at its byte i, size its bytes
// (and bit `size` that one starts behind it), least: no byte before this one may be used.  Its bytes divide
// fold_unit(q).  A lane's work.
struct FoldBlock {
  uint32_t at, bytes;                                  // the first of the two, 0 bytes: there is none
};
__device__ inline FoldBlock fold_block(uint64_t w, uint32_t size, uint32_t q, uint32_t least) {
  FoldBlock b{0, 0};
  const uint32_t unit = fold_unit(q);
  for (uint32_t bytes = q; bytes <= unit && b.bytes == 0; bytes <<= 1) {
    if (least + 2u * bytes > size) break;
    // tokens start at the same places of [at, at + bytes] and of [at + bytes, at + 2 bytes]
    uint64_t r = ~(w ^ (w >> bytes));
    for (uint32_t have = 1; have < bytes + 1u;) {
      const uint32_t step = min(have, bytes + 1u - have);
      r &= r >> step;
      have += step;
    }
    r &= w & (~0ull << least) & ((2ull << (size - 2u * bytes)) - 1ull);
    if (r) {
      b.at = (uint32_t)__builtin_ctzll(r);
      b.bytes = bytes;
    }
  }
  return b;
}

// LDS that a folded text's emission needs, in words.  Bit p of the first ones: a token starts at p, or the text ends; then, for
// each stretch, the place behind which its copies go | how many ids they are << 12.  (Three workgroups of four such waves
// fit a CU with not a block to spare: with the ranks of the words here too it was two, and runs and motifs took 90 us more.)
constexpr int kFoldStarts = kFoldBytes / 32 + 3;       // (the end, and two more that are read)
constexpr int kFoldWords = kFoldStarts + kFoldStretches;

// The ids of a folded text: those of its tokens, and each stretch's block as often as it was left out.  A wave's work;
// live, T, d: as encode_string_segmented() leaves them; out0: tokens before my positions; *total: all of them, to which the
// copies' ids are added.  Returns false, and has written nothing, if a stretch has no block that is there twice in a row.
__device__ __forceinline__ bool emit_folded(const Fold& f, uint32_t live, const uint32_t* T, uint32_t* starts, int d,
                                            uint32_t out0, int32_t* dst, uint32_t* total) {
  static_assert(kFoldStarts <= 64 && kFoldBytes < 4096, "a lane per word; fields of `copies`");
  const int lane = (int)threadIdx.x & 63;
  const uint32_t base = (uint32_t)(lane * d), n = (uint32_t)f.bytes;
  uint32_t* const copies = starts + kFoldStarts;
  wave_order();
  if (lane < kFoldStarts) starts[lane] = 0;
  wave_order();
  if (live) {
    const uint64_t mine = (uint64_t)live << (base & 31u);
    atomicOr(&starts[base >> 5], (uint32_t)mine);
    if (mine >> 32) atomicOr(&starts[(base >> 5) + 1u], (uint32_t)(mine >> 32));
  }
  if (lane == 0) atomicOr(&starts[n >> 5], 1u << (n & 31u));
  wave_order();
  const uint32_t word = lane < kFoldStarts ? starts[lane] : 0u;
  const uint32_t rank = wave_scan<OpAdd>((uint32_t)__builtin_popcount(word), 0u) - (uint32_t)__builtin_popcount(word);
  // ---- my stretch's block ----
  const uint32_t end_before = wave_shift_up(f.end, 0u);
  const bool mine = lane < f.stretches && f.out != 0;
  FoldBlock b{0, 0};
  uint64_t w = 0;
  if (mine) {
    const uint32_t i = f.first >> 5, shift = f.first & 31u;
    w = (uint64_t)__builtin_amdgcn_alignbit(starts[i + 2], starts[i + 1], shift) << 32 |
        __builtin_amdgcn_alignbit(starts[i + 1], starts[i], shift);
    b = fold_block(w, f.end - f.first, f.q, end_before > f.first ? end_before - f.first : 0u);
  }
  if (__ballot(mine && b.bytes == 0)) return false;    // uniform
  const uint32_t block = mine ? (uint32_t)(w >> (b.at + b.bytes)) & ((1u << b.bytes) - 1u) : 0u;    // the second one's tokens
  const uint32_t size = (uint32_t)__builtin_popcount(block);
  const uint32_t ids = mine ? f.out / b.bytes * size : 0u;
  const uint32_t behind = mine ? f.first + b.at + 2u * b.bytes : lane < f.stretches ? f.x : 0u;    // (ascending)
  const uint32_t upto = wave_scan<OpAdd>(ids, 0u);
  const uint32_t place = lane_read(rank, (int)(behind >> 5)) +
                         (uint32_t)__builtin_popcount(lane_read(word, (int)(behind >> 5)) & ((1u << (behind & 31u)) - 1u)) +
                         (upto - ids);
  *total += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  copies[lane] = behind | ids << 12;                   // (ids: at most 65,536)
  wave_order();
  // ---- the tokens ----
  {
    uint32_t o = out0;
    int j = 0;                                         // stretches whose copies lie before my token
    for (int i = 0; i < f.stretches; ++i) {            // uniform
      const uint32_t its_ids = (uint32_t)__builtin_amdgcn_readlane((int)ids, i);
      const bool before = (uint32_t)__builtin_amdgcn_readlane((int)behind, i) <= base;
      o += before ? its_ids : 0u;
      j += before ? 1 : 0;
    }
    for (uint32_t m = live; m; m &= m - 1u) {
      const uint32_t k = (uint32_t)__builtin_ctz(m);
      for (; j < f.stretches && (copies[j] & 0xFFFu) <= base + k; ++j) o += copies[j] >> 12;
      dst[o++] = (int32_t)(T[k * 64u + (uint32_t)lane] & kTokIdMask);
    }
  }
  // ---- the copies ----
  const uint32_t per_d = 65536u / (uint32_t)d + 1u;    // (positions are below 1,041, d at most 16: the quotient is exact)
  for (int i = 0; i < f.stretches; ++i) {              // uniform
    const uint32_t count = (uint32_t)__builtin_amdgcn_readlane((int)ids, i);
    if (count == 0) continue;
    const uint32_t tokens = (uint32_t)__builtin_amdgcn_readlane((int)size, i);
    uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)block, i);
    const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)(behind - b.bytes), i);
    int32_t* const to = dst + (uint32_t)__builtin_amdgcn_readlane((int)place, i);
    for (uint32_t c = 1; c < tokens; ++c) m = (uint32_t)lane >= c ? m & (m - 1u) : m;      // lane c: from the block's token c on
    const uint32_t at = from + (uint32_t)__builtin_ctz(m | 1u << 16);
    const uint32_t column = at * per_d >> 16;
    const uint32_t id = T[(at - column * (uint32_t)d) * 64u + min(column, 63u)] & kTokIdMask;
    uint32_t done = 0;
    if (count >= 1024u) {                              // four ids a lane and store
      uint32_t r = 4u * (uint32_t)lane % tokens;
      const uint32_t step = 256u % tokens;
      for (; done + 256u <= count; done += 256u) {
        int32_t v[4];
        uint32_t c = r;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          v[u] = (int32_t)lane_read(id, (int)c);
          c = c + 1u == tokens ? 0u : c + 1u;
        }
        __builtin_memcpy(to + done + 4u * (uint32_t)lane, v, 16);
        r += step;
        r -= r >= tokens ? tokens : 0u;
      }
    }
    uint32_t r = (done + (uint32_t)lane) % tokens;
    const uint32_t step = 64u % tokens;
    for (; done < count; done += 64u) {
      const int32_t v = (int32_t)lane_read(id, (int)r);
      if (done + (uint32_t)lane < count) to[done + (uint32_t)lane] = v;
      r += step;
      r -= r >= tokens ? tokens : 0u;
    }
  }
  return true;
}

}  // namespace bpe
