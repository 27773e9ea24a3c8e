// Splitting long strings into pieces: which string a slot belongs to, and where its piece begins and ends.  (No HIP header is
// included here, so that a host program that brings its own wave can compile this file.)
//
// No merge can cross a cut (a byte bigram that occurs at no merge junction, see table_format.h), so the two
// sides of a cut are encoded independently and their ids concatenated.  Strings longer than the piece target
// P are therefore cut near every multiple of P: the string gets ceil(len / P) "slots"; slot 0 starts at the
// string's first byte, slot i at the last cut within kCutWindow bytes before byte i*P, or is void if there is
// none (then the piece before it simply runs on).  Pieces, not strings, are what the encode kernels work on;
// their ids land in tmp_ids at the piece's own byte offset, so a string's ids are the concatenation of its
// slots' runs.
#pragma once
#include <stdint.h>

#include "table_format.h"

namespace bpe {

constexpr int kCutWindow = 128;

// A batch whose slots are all resident at once, a wave each, needs no list.  `resident`: waves of the kernel that encodes the
// pieces; rest_grid: workgroups of the one that comes after it, each of which can take kRestItems of what is left, every
// rest_grid-th item.
constexpr int kSmallSlots = 4096, kRestItems = 16;
constexpr bool small_batch_fits(int64_t slots, int64_t resident, int64_t rest_grid) {
  return slots <= kSmallSlots && slots <= resident && slots <= kRestItems * rest_grid;
}

__device__ inline uint32_t slots_of_length(int64_t len, int piece_target, int max_string) {
  // (a 32-bit division: a valid length fits, and the 64-bit one is a long software routine)
  return (len <= 0 || len > max_string) ? 1u : ((uint32_t)len + (uint32_t)piece_target - 1u) / (uint32_t)piece_target;
}

// Orders a wave's own LDS traffic (which the hardware executes in order) for the compiler.
__device__ inline void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Slots are numbered without a scan: string s's first slot is s + offsets[s] / P, and a string of ceil(len / P) slots never
// reaches the next one's.  Numbers in between that no string uses (one for every other string) are void slots too, and so are
// those before string 0's, if the offsets are a window of a longer array and do not begin with 0.
__device__ inline uint32_t slot_base(int64_t offset, int s, int piece_target) {
  return (uint32_t)s + (uint32_t)(offset >> 7) / ((uint32_t)piece_target >> 7);        // (the target is a multiple of 128)
}

// Which of the sixteen candidates q = p - 15 ... p have a cut before byte q, a bit each?  v, last: the seventeen bytes
// p - 16 ... p; m, last_m: their marks; cuts: the bit set of the cuts.
__device__ inline uint32_t cut_candidates(const uint4& v, uint32_t last, const uint4& m, uint32_t last_m, bool marked,
                                          const uint32_t* cuts) {
  const uint32_t w[5] = {v.x, v.y, v.z, v.w, last};
  uint32_t found = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t pair = (i & 3) == 3 ? __builtin_amdgcn_alignbit(w[(i >> 2) + 1], w[i >> 2], 24u) : w[i >> 2] >> (8 * (i & 3));
    found |= ((cuts[(pair >> 5) & 2047u] >> (pair & 31u)) & 1u) << i;
  }
  if (marked) {                                        // special tokens: their ends are cuts, their inside is not
    const uint32_t mark[5] = {m.x, m.y, m.z, m.w, last_m};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t two = ((i & 3) == 3 ? __builtin_amdgcn_alignbit(mark[(i >> 2) + 1], mark[i >> 2], 24u)
                                         : mark[i >> 2] >> (8 * (i & 3))) & 0xFFFFu;
      if (two) found |= 1u << i;
      if (two >> 8 == kCoverRest) found &= ~(1u << i);
    }
  }
  return found;
}
// The last cut within the kCutWindow positions up to t, or -1: a thread's own search, sixteen candidates a round; in text
// the first round nearly always finds one.  Whole waves take part, with `searching` unset where there is nothing to find.
__device__ inline int64_t last_cut(const uint8_t* bytes, const uint8_t* cover, const uint32_t* cuts, int64_t t, bool searching) {
  int64_t at = -1;
  for (int round = 0; round < kCutWindow / 16; ++round) {
    if (!__ballot(searching)) break;                   // uniform
    if (searching) {
      const int64_t p = t - 16 * round;
      uint4 v, m = make_uint4(0, 0, 0, 0);
      uint32_t last_m = 0;
      __builtin_memcpy(&v, bytes + p - 16, 16);
      if (cover) {
        __builtin_memcpy(&m, cover + p - 16, 16);
        last_m = cover[p];
      }
      const uint32_t found = cut_candidates(v, bytes[p], m, last_m, cover != nullptr, cuts);
      if (found) {
        at = p - 15 + (31 - __builtin_clz(found));
        searching = false;
      }
    }
  }
  return at;
}

// The last string whose at_or_before(s) holds, which it does up to some string (string 0 if for none), found by a whole wave:
// every round asks 64 strings at once, so 65,536 strings take three round trips instead of sixteen.  All lanes take part
// and get the result.
template <class AtOrBefore>
__device__ inline int wave_last_string(int batch, const AtOrBefore& at_or_before) {
  const int lane = threadIdx.x & 63;
  int lo = 0, n = batch;                               // the answer is one of [lo, lo + n)
  while (n > 1) {                                      // uniform; n shrinks every round
    const int step = (n + 63) >> 6;
    const int64_t i = (int64_t)lo + (int64_t)(lane + 1) * step;
    const bool upto = i < (int64_t)lo + n && at_or_before((int)i);
    const int64_t skipped = (int64_t)__builtin_popcountll(__ballot(upto)) * step;
    lo += (int)skipped;
    n = (int)min((int64_t)step, (int64_t)n - skipped);
  }
  return lo;
}

// What a wave finds in the slots g0 ... g0 + 62, a lane each; the last lane looks at one more, where their last piece may end.
// Its 64 lanes hold the strings that the slots can belong to, from s0 on, the string of slot g0.
constexpr int kListSlots = 63;
struct StepSlot {
  int64_t start;                                       // of the piece that begins in the slot, -1: none does
  int32_t len;
  int next_s0;                                         // the string of slot g0 + 63 (uniform)
};
// string_at: 64 words of LDS, the wave's own.
__device__ inline StepSlot step_slots(const uint8_t* bytes, const int64_t* offsets, int batch, const uint8_t* cover,
                                      const uint32_t* cuts, int piece_target, int max_string, uint32_t n_slots, uint32_t g0,
                                      int s0, int32_t* string_at, int32_t* slot_string, int64_t* piece_begin,
                                      int32_t* piece_len) {
  const int lane = threadIdx.x & 63;
  // my string, one of the 64 from s0 on, and the string of my slot
  const int mine = min(s0 + lane, batch - 1);
  const int64_t my_begin = offsets[mine], my_end = offsets[mine + 1];
  const uint32_t my_base = s0 + lane < batch ? slot_base(my_begin, mine, piece_target) : 0xFFFFFFFFu;
  string_at[lane] = 0;
  wave_order();
  if (lane > 0 && my_base - g0 < 64u) string_at[my_base - g0] = lane;
  wave_order();
  int owner = string_at[lane];
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(owner, d, 64);
    if (lane >= d) owner = max(owner, o);
  }
  wave_order();
  const int64_t begin = __shfl(my_begin, owner, 64), end = __shfl(my_end, owner, 64);
  const uint32_t base = (uint32_t)__shfl((int)my_base, owner, 64);
  const uint32_t g = g0 + (uint32_t)lane;
  const int i = (int)(g - base);
  const uint32_t end_slot = base + slots_of_length(end - begin, piece_target, max_string);
  const bool used = g < n_slots && g >= base && g < end_slot && end >= begin && end - begin <= max_string;
  int64_t start = last_cut(bytes, cover, cuts, begin + (int64_t)i * piece_target, used && i > 0);
  if (used && i == 0) start = begin;
  // ---- where my piece ends: at the next one of its string, or at the string's end ----
  const uint64_t pieces = __ballot(start >= 0);
  const uint64_t later = lane < 63 ? pieces & (~0ull << (lane + 1)) : 0ull;
  const int next = later ? (int)__builtin_ctzll(later) : 64;
  int64_t piece_end = __shfl(start, next & 63, 64);
  const bool beyond = start >= 0 && lane < kListSlots && (next == 64 || g0 + (uint32_t)next >= end_slot);
  if (beyond) piece_end = end;
  // (one piece at most runs on past the slots of this step)
  uint64_t runs_on = __ballot(beyond && next == 64 && end_slot > g0 + 64u);
  if (runs_on) {                                     // uniform
    const int from = (int)__builtin_ctzll(runs_on);
    const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)end_slot, from);
    const uint32_t its_base = (uint32_t)__builtin_amdgcn_readlane((int)base, from);
    const int64_t its_begin = __shfl(begin, from, 64);
    for (uint32_t h0 = g0 + 64u; h0 < last; h0 += 64u) {               // uniform
      const uint32_t h = h0 + (uint32_t)lane;
      const int64_t at = last_cut(bytes, cover, cuts, its_begin + (int64_t)(h - its_base) * piece_target, h < last);
      const uint64_t found = __ballot(at >= 0);
      const uint32_t stop = found ? h0 + (uint32_t)__builtin_ctzll(found) : last;
      if (h < stop) piece_len[h] = (int32_t)(g0 + (uint32_t)from) - (int32_t)h;
      if (found) {
        const int64_t its_end = __shfl(at, (int)__builtin_ctzll(found), 64);
        if (lane == from) piece_end = its_end;
        break;                                       // uniform
      }
    }
  }
  const int32_t len = start >= 0 ? (int32_t)(piece_end - start) : 0;
  const uint64_t before = pieces & ((1ull << lane) - 1ull);
  const int piece = before ? 63 - (int)__builtin_clzll(before) : -1;     // the piece before my slot, if it is of my string
  const bool of_my_string = piece >= 0 && g0 + (uint32_t)max(piece, 0) >= base;
  if (g < n_slots) {
    if (lane < kListSlots) {
      piece_begin[g] = start;
      slot_string[g] = i == 0 ? s0 + owner : -1;
    }
    if (start >= 0) {
      if (lane < kListSlots) piece_len[g] = len;
    } else if (used && of_my_string) {                 // (of earlier steps' pieces: theirs to say)
      piece_len[g] = piece - lane;
    } else if (!used && lane < kListSlots) {
      piece_len[g] = 0;
    }
  }
  return StepSlot{start, len, s0 + __builtin_amdgcn_readlane(owner, 63)};
}

struct SlotPiece {
  int64_t begin;
  int32_t len;                                         // -1: no piece starts in the slot
};
// The last cut within the kCutWindow positions up to t, or -1, by a whole wave: 64 candidates at a time.
__device__ inline int64_t wave_last_cut(const uint8_t* bytes, const uint8_t* cover, const uint32_t* cuts, int64_t t) {
  const int lane = threadIdx.x & 63;
  for (int round = 0; round < kCutWindow / 64; ++round) {
    const int64_t q = t - 64 * round - lane;
    const uint32_t pair = bytes[q - 1] | (uint32_t)bytes[q] << 8;
    bool cut = (cuts[pair >> 5] >> (pair & 31u)) & 1u;
    if (cover) {                                       // special tokens: their ends are cuts, their inside is not
      const uint32_t before = cover[q - 1], here = cover[q];
      cut = (cut || before != 0 || here != 0) && here != kCoverRest;
    }
    const uint64_t found = __ballot(cut);
    if (found) return t - 64 * round - (int)__builtin_ctzll(found);
  }
  return -1;
}
// The string that slot g may belong to, a wave's work: no cuts are needed for it.
struct SlotString {
  int s;
  int64_t begin, end;
};
__device__ inline SlotString slot_string_of(const int64_t* offsets, int batch, int piece_target, uint32_t g) {
  const int s = wave_last_string(batch, [&](int i) { return slot_base(offsets[i], i, piece_target) <= g; });
  return SlotString{s, offsets[s], offsets[s + 1]};
}
// The piece that starts in slot g, and what the packing kernel wants to know of the slots it covers.  A wave's work; all
// arguments are uniform.
__device__ inline SlotPiece slot_piece(const uint8_t* bytes, const SlotString& string, const uint8_t* cover,
                                       const uint32_t* cuts, int piece_target, int max_string, uint32_t g,
                                       int32_t* slot_string, int64_t* piece_begin, int32_t* piece_len) {
  const int lane = threadIdx.x & 63;
  const int s = string.s;
  const int64_t begin = string.begin, end = string.end;
  const uint32_t base = slot_base(begin, s, piece_target);
  const uint32_t end_slot = base + slots_of_length(end - begin, piece_target, max_string);
  const bool used = g >= base && g < end_slot && end >= begin && end - begin <= max_string;
  const int64_t t = begin + (int64_t)(g - base) * piece_target;
  SlotPiece piece{-1, -1};
  if (used) piece.begin = g == base ? begin : wave_last_cut(bytes, cover, cuts, t);
  if (lane == 0) {
    slot_string[g] = g == base ? s : -1;
    piece_begin[g] = piece.begin;
    if (!used) piece_len[g] = 0;                       // (of a void slot that a piece runs over: the piece's wave)
  }
  if (piece.begin < 0) return piece;
  int64_t piece_end = end;
  if (g + 1u < end_slot) {
    int64_t next = wave_last_cut(bytes, cover, cuts, t + piece_target);
    for (uint32_t h0 = g + 1u; next < 0 && h0 < end_slot; h0 += 64u) {   // a slot a lane
      const uint32_t h = h0 + (uint32_t)lane;
      const int64_t at = last_cut(bytes, cover, cuts, begin + (int64_t)(h - base) * piece_target, h < end_slot);
      const uint64_t found = __ballot(at >= 0);
      const uint32_t stop = found ? h0 + (uint32_t)__builtin_ctzll(found) : end_slot;
      if (h < stop) piece_len[h] = (int32_t)g - (int32_t)h;
      if (found) next = __shfl(at, (int)__builtin_ctzll(found), 64);
    }
    if (next >= 0) piece_end = next;
  }
  piece.len = (int32_t)(piece_end - piece.begin);
  if (lane == 0) piece_len[g] = piece.len;
  return piece;
}

}  // namespace bpe
