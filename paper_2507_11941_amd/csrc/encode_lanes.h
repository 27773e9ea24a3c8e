// One lane per segment: the encoder for work items of up to 2 KiB whose segments are short.
//
// A string falls apart at its cuts -- byte bigrams that lie at no merge junction, see table_format.h -- into
// segments that Algorithm 1 processes without any interaction; with word-like text a segment is a word of a
// few bytes.  Most of them are one token of the vocabulary and are looked up as a whole (word_table.h).  In the others
// there is nothing for 64 lanes to share, so every lane takes a whole segment and runs Algorithm 1 on it literally: find
// the lowest-rank pair (left-most on ties), replace it by its merged token, look up the two pairs the new token forms
// (section 4.2's steps, one lane wide), until no pair of the segment is in the table.  The wave as a whole still works
// on one item (section 4.3: one block per string), and a lane that finishes its segment takes the item's next one,
// longer segments first, so the lanes stay busy whatever the mix of segment lengths.
//
//   cuts     lane t holds bytes 16 t ... 16 t + 15 of the item (one wide load), asks a bit set of all byte bigrams in LDS
//            where they are cut, and leaves the segments' first positions as a bitmap, then as a list -- without the
//            segments of one byte, which are a token as they are, where those are many.
//   words    segment-parallel, 64 at a time and three such batches in flight: the segment's bytes are its key; two
//            dependent table reads say which token it is, if it is one.
//   list     the other segments, the "jobs", sorted by length, longest first: a counting sort with one LDS counter per
//            length.  Handing the long segments out first is what keeps the lanes level at the end; up to 64 jobs are
//            not sorted, every lane has one at once (64 strings of 4 KiB: 0.4 us).  Only they get a place in the array of
//            tokens and pair values (the "arena").
//   merge    segment-parallel, as above; a lane keeps its segment's liveness as a 32-bit mask, so a segment
//            may have at most 32 bytes.  A string with a longer segment is not encoded here: the kernel hands
//            it to the wave-per-item encoder of encode_segmented.h, which has no such limit.  (An item is one
//            string, a piece of one, or a group of short ones; of a group only such strings are handed on.)
//   emit     a bitmap of the item says where tokens start; the bits before one are its place in the output (section 4.3's
//            compaction).  Words and jobs segment-parallel, single bytes position-parallel.
//
// list to emit run over as many jobs at a time as the arena and the list hold: in words, all of the item's.
//
// What bounds it is instruction issue: some 2,100 vector and 550 scalar instructions per KiB of text, of which the merge
// loop is two fifths, on four waves a SIMD.  With every segment going through the merges, one item of 1 KiB a wave
// (14.9 trips of the loop per KiB instead of 6.8), the 65,536 documents of the throughput workload took 1,480 us in this
// kernel; they take 977, and the whole call 1,066 instead of 1,659 (1,053 since no claim makes a loop over the lanes, see wave_claim).
//
// Of text that is not words most look-ups find nothing and cost what they cost, and its jobs do not fit the arena at once.
// 32 MiB in strings of 4 KiB, whole call, all segments merged / single bytes listed and looked up like the others, the arena
// filled to the brim and the rest in a part of its own / now: bytes at random, 100k rows 281 / 453 / 241 us; digits and
// letters of a hexadecimal dump, 32k rows 303 / 405 / 332; text of a larger table's words under 1k rows 254 / 396 / 305;
// words of no table, 100k rows 314 / 367 / 371; words, 100k rows 312 / 241 / 239.  (Single bytes four positions a lane instead
// of a row at a time: 3 to 4 % off the third, but 128 registers, and 0.4 % more for words and 1.8 % for runs and motifs.)
#pragma once
#include "encode_segmented.h"

namespace bpe {

constexpr int kLaneSegmentMax = 32;             // positions a lane's liveness mask covers
constexpr int kLaneBatches = 3;                 // batches of 64 segments whose look-ups are in flight together
constexpr uint32_t kLaneChunk = 4;              // work items a wave claims at a time (1: 3.4 ms on 270,000 pieces of
                                                // 1 KiB, 2: 2.2, 4: 2.1, 8: 2.1, when all their segments were merged);
                                                // twice as many when the list holds 32 or more items per wave

// What the lanes keep of a segment is one word for each of its positions.  It is the value of the pair that begins there,
// with the position in its lowest bits, so that the lowest value says where it is:
//   bits 0..4 position in the segment, 5 and 6 the merged token can be a left / right operand, 7..26 rank
// or, behind a token that merges have made (the position after its first is always a dead one), that token's word:
//   bits 0..19 id, 20 and 21 it can be a left / right operand, 31 set (above every pair)
// A token that no merge has made is its byte, which is still in the text.
constexpr uint32_t kLaneNoPair = 0xFFFFFFFFu;
constexpr uint32_t kLaneNoTag = 0xF8000000u;    // no slot's tag: fingerprints have 27 bits, an empty slot is all ones
constexpr uint32_t kLaneInvalid = 0xFFFFEu << 7;       // values from here on are no pair (ranks stay below 0xFFFFE)
constexpr uint32_t kLaneCanLeft = 1u << 20, kLaneCanRight = 1u << 21;

__device__ inline uint32_t lane_value(uint32_t v, uint32_t position) {
  static_assert(kFlagLeft == 1u << 10 && kFlagRight == 1u << 11 && kRankShift == 12, "flag positions");
  return ((v >> 10) << 5) | position;
}
__device__ inline uint32_t lane_merged_word(uint32_t lv) {
  return ((lv >> 7) + (256u | 1u << 31)) | ((lv & 0x60u) << 15);
}
// (a byte that no row can use costs a look-up that finds nothing; asking for its bits costs another LDS round trip)
__device__ inline uint32_t lane_byte_word(uint32_t byte) { return byte | kLaneCanLeft | kLaneCanRight; }

constexpr uint32_t kRecNone = 1u << 31;         // what becomes of a segment: its token's number, or this: it is not one token

// LDS of a workgroup, in 32-bit words: read-only, shared by its waves.
struct LaneShared {
  static constexpr int kCuts = 0;                                       // bit a + 256 b: bytes a, b have a cut between them
  static constexpr int kMasks = kCuts + 2048;                           // [16][4] first l bytes of a key
  static constexpr int kWords = kMasks + 64;
};
// Shape of a workgroup, and the LDS of one of its waves.  WAVES: they take items of their own; BYTES: an item's capacity;
// LIST: segments listed at a time; JOBS: those that go through the merges at a time; ARENA: the bytes of those, in fours.  What bounds
// the number of waves is LDS, and what bounds the kernel is how many waves there are to wait at once: 65,536 documents take
// 1,554 us with 8 waves a CU, 1,379 with 10, 1,232 with 12 (that was with the tokens in a second array beside V) and 1,107
// with the 16 that one array leaves room for.  Twice as long an item takes less than half as many trips of the merge loop
// for each of its bytes (the longest chain of merges is 10 long in either): the same batch in items of 1 KiB took 1,443
// instead of 1,232.  A small batch wants each piece of text to have a wave; its items of 1 KiB fit the arena whatever they
// hold (1,024 strings of 1 KiB of words of no table: 35 us in two parts, 28 in one).
template <int BYTES, int WAVES, int LIST, int JOBS, int ARENA, int AT_LEAST>
struct LaneShape {
  static constexpr int kBytes = BYTES, kWaves = WAVES, kListed = LIST, kMostJobs = JOBS, kArena = ARENA;
  static constexpr int kText = 0;                                       // the item's bytes; a key's words reach beyond them
  static constexpr int kStrings = kText + BYTES / 4 + 8;                // (groups) bit p: a string starts at p
  static constexpr int kTokens = kStrings + BYTES / 32;                 // bit p: a token starts at p
  static constexpr int kRanks = kTokens + BYTES / 32;                   // uint16 tokens before each word of kTokens
  static constexpr int kHeads = kRanks + BYTES / 64;                    // uint16 last start in the words before each of kStrings
  static constexpr int kList = kHeads + BYTES / 64;                     // uint16 segments: first position | (length - 1) << 11
  static constexpr int kJobs = kList + LIST / 2;                        // the jobs sorted: the same, and the arena's places up to it << 16
  static constexpr int kHist = kJobs + JOBS;                            // jobs of each length, then list bases
  static constexpr int kV = (kHist + 32 + 3) / 4 * 4;                   // a word for every arena position
  static constexpr int kIdle = kV + ARENA;                              // what a lane without a segment reads and writes
  static constexpr int kEnd = kIdle + 4;
  // before the arena is used:
  static constexpr int kStarts = kV;                                    // bit p: a segment starts at p, or the item ends
  static constexpr int kFound = kV;                                     // what becomes of a segment
  static constexpr int kWords = ((kEnd > AT_LEAST ? kEnd : AT_LEAST) + 3) / 4 * 4;
  static constexpr size_t kLdsBytes = lds_blocks(sizeof(uint32_t) * (LaneShared::kWords + WAVES * kWords));
  static_assert(kText % 4 == 0 && ARENA % 4 == 0 && LaneShared::kWords % 4 == 0, "wide loads and stores");
  static_assert(ARENA <= 2048 && BYTES <= 2048 && BYTES % 1024 == 0 && LIST % 64 == 0 && LIST <= 1024 && JOBS % 64 == 0,
                "fields of the packed words; a lane per word of the bitmap");
  static_assert(LIST <= ARENA && BYTES / 32 + 4 <= ARENA, "what shares a place fits it");
  static_assert(kLdsBytes <= 160 * 1024, "one workgroup a CU");
};
using LargeItems = LaneShape<kGroupBytes, 16, 448, 256, 1168, 0>;
using SmallItems = LaneShape<kMemberBytes, 16, 256, 256, 1536, 0>;
// (the arrays of the one-wave encoder that takes a string over)
constexpr int kOtherWords = encode_array_words<1, 16, false, true>() + encode_exchange_words<1>();
using InlineItems = LaneShape<kMemberBytes, 12, 256, 256, 1536, kOtherWords>;

__device__ inline uint32_t mbcnt64(uint64_t mask) {                     // set bits of mask below my lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
// A look-up in the merge table on its way: two start at the end of every trip of the merge loop.
struct LaneProbe {
  uint4 q;                                             // the home bucket: two slots of {value, tag}
  uint32_t bucket, tag;                                // kLaneNoTag: no look-up
};
__device__ inline void lane_probe_start(const DeviceTable& t, uint32_t xw, uint32_t yw, LaneProbe& f) {
  static_assert(kLaneCanLeft << 1 == kLaneCanRight, "one bit beside the other");
  f.tag = kLaneNoTag;
  if ((xw << 1) & yw & kLaneCanRight) {                // the left token can be a left operand, the right one a right one
    const Placement pl = place_pair(xw & kTokIdMask, yw & kTokIdMask, t.log2_buckets);
    f.bucket = pl.bucket;
    f.tag = slot_tag(pl.fingerprint, 0);
    f.q = t.buckets[pl.bucket];
  }
}
// Both values, kNoRank where there is no such row.  The wait is spelled out: where the first use of a load lies in a
// branch, the compiler waits at the register's next write, and that is where the next trip starts its loads -- each then
// waited for the one before it.
__device__ inline void lane_probe_finish(const DeviceTable& t, const LaneProbe& a, const LaneProbe& b, uint32_t& ra, uint32_t& rb) {
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
  ra = match_bucket(a.q, a.tag);
  rb = match_bucket(b.q, b.tag);
  // a pair that is not in its full home bucket may have been displaced, as far as the bucket's spare bits say
  uint32_t left_a = ra == kNoRank && a.q.w != kNoRank && a.tag != kLaneNoTag ? bucket_reach(a.q.x, a.q.z) : 0u;
  uint32_t left_b = rb == kNoRank && b.q.w != kNoRank && b.tag != kLaneNoTag ? bucket_reach(b.q.x, b.q.z) : 0u;
  uint32_t d = 1;
  while (__ballot((left_a | left_b) != 0)) {           // one read a lane and trip
    if (left_a | left_b) {
      const bool first = left_a != 0;
      const uint32_t tag = (first ? a.tag : b.tag) | (d << kTagDisplacementShift);
      const uint32_t found = match_bucket(t.buckets[(first ? a.bucket : b.bucket) ^ d], tag);
      const bool over = found != kNoRank || d >= (first ? left_a : left_b);
      if (first) ra = found; else rb = found;
      if (over && first) left_a = 0;
      if (over && !first) left_b = 0;
      d = over ? 1u : d + 1u;
    }
  }
}

// Encodes item s -- n bytes from `begin` on (both uniform) -- if all its segments fit a lane; returns 1 (and
// has written nothing to global memory) if one does not, else 0.  lds: this wave's words of the shape L; shared: the
// workgroup's LaneShared.  GROUPS: the item is the `members` strings from s on, at most 64, which lie one after the other
// in those bytes: a string's first byte starts a segment, and each string gets its own count.  The result has a
// bit for every string with a segment that fits no lane; the others are encoded all the same, and if there is such a
// string, each one's ids lie at its own place in tmp_ids instead of one after the other.  (100,000 rows of up to 60 bytes,
// one in twenty with such a segment: 153 us.  With the whole group given away, five rows in six went to the wave-per-item
// encoder: 1,029 us; with each row an item of its own 728; both when all segments were merged and this took 183.)
template <class L, bool SPECIAL, bool GROUPS, bool ALONE>
__device__ __forceinline__ uint64_t encode_item_lanes(const EncodeParams& p, int s, int64_t begin, int n, int members,
                                                      uint32_t* lds, const uint32_t* shared) {
  const int lane = (int)threadIdx.x & 63;
  const DeviceTable& tab = p.table;
  uint32_t* const text = lds + L::kText;
  uint32_t* const starts = lds + L::kStarts;
  uint32_t* const strings = lds + L::kStrings;
  uint32_t* const tokens = lds + L::kTokens;
  uint16_t* const ranks = (uint16_t*)(lds + L::kRanks);
  uint16_t* const heads = (uint16_t*)(lds + L::kHeads);
  uint16_t* const list = (uint16_t*)(lds + L::kList);
  uint32_t* const jobs = lds + L::kJobs;
  uint32_t* const hist = lds + L::kHist;
  uint32_t* const V = lds + L::kV;

  if (n <= 0 || n > L::kBytes) {                  // uniform; too long only if max_len was wrong
    if constexpr (GROUPS) {
      for (int i = lane; i < members; i += 64) p.counts[s + i] = 0;
    } else {
      if (lane == 63) p.counts[s] = 0;
    }
    return 0;
  }
  __builtin_amdgcn_s_setprio(3);                       // (the load phase too is a chain of round trips, and the
                                                       // sooner its loads go out the better)

  // ---- cuts: where the segments start ----
  constexpr int kPasses = L::kBytes / 1024;       // a wave holds 1 KiB at a time
  uint4 q[kPasses], marks[kPasses];
#pragma unroll
  for (int pass = 0; pass < kPasses; ++pass) {
    const int at = 1024 * pass + 16 * lane;
    q[pass] = marks[pass] = make_uint4(0, 0, 0, 0);
    if (at < n) {
      q[pass] = load_16_bytes(p.bytes + begin, at, begin, p.total_bytes - begin);
      if constexpr (SPECIAL) marks[pass] = load_16_bytes(p.cover + begin, at, begin, p.total_bytes - begin);
    }
  }
  int from = n, to = n;                                // (groups) where string `lane` begins and ends in the item
  if constexpr (GROUPS) {
    if (lane < members) from = (int)min(max(p.member_begin[s + lane] - begin, (int64_t)0), (int64_t)n);
    to = (int)lane_read((uint32_t)from, min(lane + 1, 63));
    if (lane + 1 >= members) to = n;
    if (lane < L::kBytes / 32) strings[lane] = 0;
    wave_order();
    if (from < n) atomicOr(&strings[from >> 5], 1u << (from & 31));
    wave_order();
  }
  bool any_marked = false;                             // (special tokens) uniform
  {
    uint32_t cut_before = 1, marked_before = 0;        // of the pass's first byte (uniform); the item starts a segment
#pragma unroll
    for (int pass = 0; pass < kPasses; ++pass) {
      if (1024 * pass < n) {                           // uniform
        const int at = 1024 * pass + 16 * lane;
        const uint4 v = q[pass];
        *(uint4*)(text + 256 * pass + 4 * lane) = v;
        uint32_t after = wave_shift_down(v.x, 0u);     // the bytes after mine
        if (pass + 1 < kPasses) {
          const uint32_t wrap = (uint32_t)__builtin_amdgcn_readlane((int)q[pass + 1 < kPasses ? pass + 1 : pass].x, 0);
          after = lane == 63 ? wrap : after;
        }
        const uint32_t w[5] = {v.x, v.y, v.z, v.w, after};
        uint32_t ends = 0;                             // bit j: a cut after my byte j
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          // bytes j and j + 1 in the low 16 bits, what lies above them is not looked at
          const uint32_t pair = (j & 3) == 3 ? __builtin_amdgcn_alignbit(w[(j >> 2) + 1], w[j >> 2], 24u)
                                             : w[j >> 2] >> (8 * (j & 3));
          const uint32_t bits = shared[LaneShared::kCuts + ((pair >> 5) & 2047u)];
          ends |= __builtin_amdgcn_ubfe(bits, pair & 31u, 1u) << j;
        }
        const uint32_t ends_before = wave_shift_up(ends, 0u);            // (all lanes: not inside a branch)
        uint32_t begins = (ends << 1) | (lane == 0 ? cut_before : ends_before >> 15);
        if constexpr (SPECIAL) {
          // an occurrence of a special token is one token on its first byte and nothing on the others: every marked
          // byte is a segment of its own
          const uint4 m = marks[pass];
          uint32_t marked = 0, inside = 0;             // (inside: no token)
          if (__ballot((m.x | m.y | m.z | m.w) != 0)) {
            any_marked = true;
            // (a mark's top bit, or the one below it, says which kind it is, four marks at a time: one by one the kernel took 340
            // us on 54 MB of separated documents instead of 329)
            static_assert(kCoverFirst == 0x80u && kCoverRest == 0x40u && kCoverIndex == 0x3Fu, "bits of a mark");
            const uint32_t mw[4] = {m.x, m.y, m.z, m.w};
            uint32_t firsts = 0;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
              firsts = firsts << 4 | __builtin_amdgcn_udot4((mw[j] >> 7) & 0x01010101u, 0x08040201u, 0u, false);
              inside = inside << 4 | __builtin_amdgcn_udot4((mw[j] >> 6) & 0x01010101u, 0x08040201u, 0u, false);
            }
            marked = firsts | inside;
            if (at < n && n - at < 16) marked &= (1u << (n - at)) - 1u;      // (the next string's, or none)
          }
          ((uint16_t*)tokens)[64 * pass + lane] = (uint16_t)~inside;
          const uint32_t mine_before = wave_shift_up(marked, 0u);
          begins |= marked | (marked << 1) | (lane == 0 ? marked_before : mine_before >> 15);
          marked_before = (uint32_t)__builtin_amdgcn_readlane((int)marked, 63) >> 15;
        }
        cut_before = ((uint32_t)__builtin_amdgcn_readlane((int)ends, 63) >> 15) & 1u;
        if constexpr (GROUPS) begins |= ((const uint16_t*)strings)[64 * pass + lane];
        const int here = n - at;                       // bytes of the item from my first one on
        begins &= here >= 16 ? 0xFFFFu : here > 0 ? (1u << here) - 1u : 0u;
        if (here >= 0 && here < 16) begins |= 1u << here;                  // the item's end
        ((uint16_t*)starts)[64 * pass + lane] = (uint16_t)begins;
        // (the words after the pass's; the end itself if it lies there)
        if (lane < 4) ((uint16_t*)starts)[64 * (pass + 1) + lane] = (uint16_t)(lane == 0 && n == 1024 * (pass + 1));
      }
    }
  }
  wave_order();
  __builtin_amdgcn_s_setprio(0);

  // ---- segments that no lane can take: more than 32 positions from a start to the next (nothing has left LDS) ----
  const int n_words = (n + 31) >> 5;                   // words of the bitmap, a lane each (uniform)
  uint64_t left = 0;                                   // strings that are not encoded here (uniform)
  const uint32_t my_starts = lane < n_words ? starts[lane] : 0u;         // (the item's end among them)
  const uint32_t next = lane < n_words ? starts[lane + 1] : 0u;
  uint32_t segments = my_starts;                       // first positions of the segments that are encoded here
  if (32 * lane + 31 >= n && lane < n_words && (n & 31)) segments &= (1u << (n & 31)) - 1u;
  {
    const int top = 32 * lane + 31 - (int)__builtin_clz(my_starts | 1u);   // the word's last start
    const bool empty = lane < n_words && my_starts == 0;
    const bool gap = my_starts != 0 && next != 0 && top < n &&
                     __builtin_clz(my_starts) + __builtin_ctz(next | 0x80000000u) + 1 > kLaneSegmentMax;
    uint64_t too_long = __ballot(empty || gap);
    if (too_long) {                                    // uniform
      if constexpr (!GROUPS) return 1;
      // The strings that hold one: lane m asks for string m.  They get no tokens below.
      const int inside = empty ? 32 * lane : top;
      for (; too_long; too_long &= too_long - 1ull) {  // uniform
        const int at = __builtin_amdgcn_readlane(inside, (int)__builtin_ctzll(too_long));
        left |= __ballot(from <= at && at < to);
      }
      for (uint64_t m = left; m; m &= m - 1ull) {      // uniform
        const int lo = max(__builtin_amdgcn_readlane(from, (int)__builtin_ctzll(m)) - 32 * lane, 0);
        const int hi = min(__builtin_amdgcn_readlane(to, (int)__builtin_ctzll(m)) - 32 * lane, 32);
        if (lo < hi) segments &= ~((hi >= 32 ? 0xFFFFFFFFu : (1u << hi) - 1u) & (0xFFFFFFFFu << lo));
      }
    }
  }
  const uint32_t follows = __builtin_amdgcn_alignbit(next, my_starts, 1u);   // bit p: a segment, or nothing, starts at p + 1
  const uint32_t multi = segments & ~follows;          // segments of two bytes or more; the others are a token each as they are
  const uint64_t any_multi = __ballot(multi != 0);

  int32_t* const dst = ALONE && p.out_offsets ? p.out_ids : p.tmp_ids + begin;
  // Single bytes all (blank lines, padding that no row joins): their ids are the bytes.  (64 strings of 64 KiB of spaces: 16 us,
  // as segments 48.)
  if (!any_multi && !any_marked && !left) {            // uniform
    for (int o = lane; o < n; o += 64) dst[o] = (int32_t)((text[o >> 2] >> (8 * (o & 3))) & 0xFFu);
    if constexpr (GROUPS) {
      if (lane < members) {
        p.counts[s + lane] = to - from;
        if (p.group_ids) p.group_ids[s + lane] = lane == 0 ? n : 0;
      }
    } else {
      if (lane == 63) p.counts[s] = n;
    }
    wave_order();
    return 0;
  }
  // ---- where tokens start: at the segments' first bytes, and wherever the merges leave one ----
  uint32_t singles = segments & follows;
  {
    uint32_t first_tokens = segments;
    if constexpr (SPECIAL) {
      const uint32_t not_inside = lane < n_words ? tokens[lane] : 0u;
      singles &= not_inside;
      first_tokens &= not_inside;
    }
    if (lane < L::kBytes / 32) tokens[lane] = first_tokens;
  }
  if constexpr (GROUPS) {
    if (left) {                                        // uniform: strings at their own places
      const uint32_t my_heads = lane < L::kBytes / 32 ? strings[lane] : 0u;
      const uint32_t upto = wave_scan<OpMax>(my_heads ? 32u * (uint32_t)lane + 31u - (uint32_t)__builtin_clz(my_heads) : 0u, 0u);
      const uint32_t before = wave_shift_up(upto, 0u);
      if (lane < L::kBytes / 32) heads[lane] = (uint16_t)before;
    }
  }
  wave_order();
  uint32_t my_tokens = 0, my_rank = 0, total = 0;      // word `lane` of the bitmap, the tokens before it, all (uniform)
  auto count_tokens = [&]() {
    wave_order();
    my_tokens = lane < L::kBytes / 32 ? tokens[lane] : 0u;
    const uint32_t upto = wave_scan<OpAdd>((uint32_t)__builtin_popcount(my_tokens), 0u);
    my_rank = upto - (uint32_t)__builtin_popcount(my_tokens);
    total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    if (lane < L::kBytes / 32) ranks[lane] = (uint16_t)my_rank;
    wave_order();
  };
  // tokens before position `at`, which is in the item
  auto rank_of = [&](uint32_t at) {
    return (uint32_t)ranks[at >> 5] + (uint32_t)__builtin_popcount(tokens[at >> 5] & ((1u << (at & 31u)) - 1u));
  };
  // (strings at their own places) what the place of a token of the string that holds position `at` lacks to it
  auto lack_of = [&](uint32_t at) {
    const uint32_t here = strings[at >> 5] & ((2u << (at & 31u)) - 1u);
    const uint32_t head = here ? (at | 31u) - (uint32_t)__builtin_clz(here) : heads[at >> 5];
    return head - rank_of(head);
  };
  // Few single bytes (one or two in a word here and there) are listed with the others: a look-up batch has room for them, and
  // a pass of their own costs a wave that is alone half a microsecond.
  const bool few = !__ballot(__builtin_popcount(singles) > 2);           // uniform
  const uint32_t listed = few ? multi | singles : multi;
  if (few) singles = 0;
  const uint32_t my_listed = (uint32_t)__builtin_popcount(listed);
  const uint32_t all_upto = wave_scan<OpAdd>(my_listed, 0u);
  uint32_t listed_before = 0;                          // segments of earlier lists (uniform)
  const bool any_listed = __ballot(listed != 0) != 0;  // uniform
  if (!any_listed) count_tokens();
  for (int word0 = any_listed ? 0 : n_words; word0 < n_words;) {         // (one list, unless there are very many segments)
    // ---- list of the segments that start in words word0 ... word1 - 1 ----
    const uint64_t in_list = __ballot(lane >= word0 && lane < n_words && all_upto - listed_before <= (uint32_t)L::kListed);
    const int word1 = word0 + (int)__builtin_popcountll(in_list);          // (at least one more: a word has 18 at most)
    const uint32_t listed_upto = (uint32_t)__builtin_amdgcn_readlane((int)all_upto, word1 - 1);
    const int n_listed = (int)(listed_upto - listed_before);
    {
      uint32_t at = all_upto - my_listed - listed_before;
      uint32_t m = lane >= word0 && lane < word1 ? listed : 0u;
      while (__ballot(m != 0)) {
        if (m) {
          const uint32_t bit = (uint32_t)__builtin_ctz(m);
          const uint32_t window = __builtin_amdgcn_alignbit(next >> 1, follows, bit);    // (its next start is among these)
          list[at++] = (uint16_t)((32u * (uint32_t)lane + bit) | ((uint32_t)__builtin_ctz(window | 0x80000000u) << 11));
        }
        m &= m - 1u;
      }
    }
    wave_order();
    word0 = word1;
    listed_before = listed_upto;

    // ---- words: which segments are one token ----
#pragma unroll 1
    for (int base = 0; base < n_listed; base += 64 * kLaneBatches) {     // uniform
      uint32_t k[kLaneBatches][4], len[kLaneBatches], tag[kLaneBatches], at[kLaneBatches], mark[kLaneBatches];
      uint4 bucket[kLaneBatches], key[kLaneBatches];
#pragma unroll
      for (int r = 0; r < kLaneBatches; ++r) {
        const uint32_t e = list[min(base + 64 * r + lane, n_listed - 1)];
        if constexpr (SPECIAL) at[r] = e & 2047u;
        len[r] = (e >> 11) + 1u;
        const uint32_t* const word = text + ((e & 2047u) >> 2);
        const uint32_t shift = 8u * (e & 3u);
        const uint4 mask = *(const uint4*)(shared + LaneShared::kMasks + 4 * min(len[r], (uint32_t)kWordBytes));
        k[r][0] = __builtin_amdgcn_alignbit(word[1], word[0], shift) & mask.x;
        k[r][1] = __builtin_amdgcn_alignbit(word[2], word[1], shift) & mask.y;
        k[r][2] = __builtin_amdgcn_alignbit(word[3], word[2], shift) & mask.z;
        k[r][3] = (__builtin_amdgcn_alignbit(word[4], word[3], shift) & mask.w) | (len[r] << 24);
      }
#pragma unroll
      for (int r = 0; r < kLaneBatches; ++r) {
        tag[r] = 0;
        bucket[r] = make_uint4(kWordNone, kWordNone, kWordNone, kWordNone);
        if (base + 64 * r < n_listed) {                // uniform
          const uint32_t hash = word_hash(k[r][0], k[r][1], k[r][2], k[r][3]);
          tag[r] = word_tag(hash);
          if (len[r] - 2u <= (uint32_t)kWordBytes - 2u)
            bucket[r] = tab.word_buckets[word_bucket(hash, tab.log2_word_buckets)];
        }
        if constexpr (SPECIAL) {
          mark[r] = 0;
          if (any_marked && len[r] == 1u) mark[r] = p.cover[begin + at[r]];
        }
      }
#pragma unroll
      for (int r = 0; r < kLaneBatches; ++r) {
        // (at most one slot of a bucket has the tag; an empty one leaves all ones in the id's bits at best)
        tag[r] = min(min(bucket[r].x ^ tag[r], bucket[r].y ^ tag[r]), min(bucket[r].z ^ tag[r], bucket[r].w ^ tag[r]));
        key[r] = make_uint4(0, 0, 0, 0);               // (no key: a key has a length)
        if (tag[r] < (1u << kWordIdBits) - 1u) key[r] = tab.word_keys[tag[r]];
      }
#pragma unroll
      for (int r = 0; r < kLaneBatches; ++r) {
        if (base + 64 * r < n_listed) {                // uniform
          const bool same = ((key[r].x ^ k[r][0]) | (key[r].y ^ k[r][1]) | (key[r].z ^ k[r][2]) | (key[r].w ^ k[r][3])) == 0;
          uint32_t what = same ? tag[r] : kRecNone;
          if (len[r] == 1u) {
            what = k[r][0];
            if constexpr (SPECIAL)
              if (mark[r]) what = p.special_base + (mark[r] & kCoverIndex);
          }
          lds[L::kFound + base + 64 * r + lane] = what;
        }
      }
    }
    wave_order();
    // ---- the others ("jobs") need merges, and a place in the arena: four words or more, whole fours ----
    constexpr int kBatches = L::kListed / 64;
    // found: what becomes of segment 64 r + lane.  job: list entry of the r-th segment that the lane has, and the places up to
    // it << 16; 0 if it is no job.
    const int each = (n_listed + 63) >> 6;             // uniform
    uint32_t found[kBatches], job[kBatches];
#pragma unroll
    for (int r = 0; r < kBatches; ++r) found[r] = job[r] = 0;
    uint32_t all_places = 0, part = 0, n_jobs = 0;     // uniform
    for (int by_lane = 1, by_r = 64;;) {               // uniform
#pragma unroll
      for (int r = 0; r < kBatches; ++r) {             // (all reads go out before the first is waited for)
        if (r >= each) break;                          // uniform
        const int i = by_lane * lane + by_r * r;
        const uint32_t what = lds[L::kFound + i], e = list[i];
        found[r] = by_lane == 1 ? what : found[r];
        const uint32_t is_job = (uint32_t)((int)what >> 31);             // (kRecNone or a token's number)
        job[r] = i < n_listed ? e & is_job : 0u;                         // (a segment has a length)
      }
      uint32_t mine = 0;                               // places | jobs << 16
#pragma unroll
      for (int r = 0; r < kBatches; ++r) {
        if (r >= each) break;                          // uniform
        if (job[r]) {
          mine += (((job[r] >> 11) + 4u) & ~3u) + 0x10000u;
          job[r] |= mine << 16;
        }
      }
      const uint32_t upto = wave_scan<OpAdd>(mine, 0u);
#pragma unroll
      for (int r = 0; r < kBatches; ++r) {
        if (r >= each) break;                          // uniform
        if (job[r]) job[r] += (upto - mine) << 16;
      }
      const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
      part = all_places = all & 0xFFFFu;
      n_jobs = all >> 16;
      // As many as the arena and the jobs' list hold at a time: all of the item's, in text.  Else in parts of about the
      // same size, for each part ends with some lanes idle, a small one as much as a large one; and parts of the text, so
      // that what lies before a part is known when it is written: the lanes' segments are neighbours then.
      if (all_places <= (uint32_t)L::kArena && n_jobs <= (uint32_t)L::kMostJobs) break;
      const uint32_t most = min(n_jobs > (uint32_t)L::kMostJobs ? 4u * (uint32_t)L::kMostJobs : ~0u, (uint32_t)L::kArena);
      const uint32_t parts = (all_places + most - 1u) / most;
      part = min(all_places / parts + (uint32_t)kLaneSegmentMax, most);
      if (by_r == 1 || each == 1) break;
      by_lane = each;
      by_r = 1;
    }
    auto write_words = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < kBatches; ++r) {
        if (r >= each) break;                            // uniform
        if (64 * r + lane < n_listed && found[r] != kRecNone) {
          const uint32_t at = list[64 * r + lane] & 2047u;
          uint32_t o = rank_of(at);
          if constexpr (GROUPS)
            if (left) o += lack_of(at);
          dst[o] = (int32_t)found[r];
        }
      }
    };
    if (!all_places) {                                 // uniform
      count_tokens();
      write_words();
    }
    for (uint32_t done = 0; done < all_places;) {      // uniform: places of the parts before
      wave_order();
      uint32_t upto_part = all_places;                 // uniform
      // where a job begins in the arena: whole fours
      auto place_of = [&](uint32_t e) { return (e >> 16) - done - ((((e >> 11) & 31u) + 4u) & ~3u); };
      if (n_jobs <= 64u && part == all_places) {       // uniform: a lane for each at once, in whatever order
        uint32_t before = 0;
#pragma unroll
        for (int r = 0; r < kBatches; ++r) {
          if (r >= each) break;                        // uniform
          const uint64_t mine = __ballot(job[r] != 0);
          if (job[r]) jobs[before + mbcnt64(mine)] = job[r];
          before += (uint32_t)__builtin_popcountll(mine);
        }
        wave_order();
      } else {
        // ---- list: longest first (counting sort over the 31 possible lengths) ----
        if (lane < 32) hist[lane] = 0;
        wave_order();
        uint32_t place[kBatches], mine = 0, last = done;
#pragma unroll
        for (int r = 0; r < kBatches; ++r) place[r] = 0;
#pragma unroll
        for (int r = 0; r < kBatches; ++r) {
          if (r >= each) break;                        // uniform
          if ((job[r] >> 16) - done - 1u < part) {
            place[r] = atomicAdd(&hist[31u - ((job[r] >> 11) & 31u)], 1u);                       // among those of its length
            ++mine;
            last = job[r] >> 16;
          }
        }
        if (part < all_places) {                       // uniform
          n_jobs = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan<OpAdd>(mine, 0u), 63);
          upto_part = wave_reduce<OpMax>(last);
        }
        wave_order();
        {
          const uint32_t mine = lane < 32 ? hist[lane] : 0u;
          const uint32_t inc = wave_scan<OpAdd>(mine, 0u);
          wave_order();
          if (lane < 32) hist[lane] = inc - mine;      // where the segments of length 32 - lane start
        }
        wave_order();
#pragma unroll
        for (int r = 0; r < kBatches; ++r) {
          if (r >= each) break;                        // uniform
          if ((job[r] >> 16) - done - 1u < part)
            jobs[hist[31u - ((job[r] >> 11) & 31u)] + place[r]] = job[r];
        }
        wave_order();
      }
      {
        // ---- in the arena: byte-level pre-tokenisation (section 4.1) and the initial pair values ----
#pragma unroll 1
        for (uint32_t j0 = 0; j0 < n_jobs; j0 += 64) { // uniform
          const uint32_t j = j0 + (uint32_t)lane;
          const uint32_t e = jobs[min(j, n_jobs - 1u)];
          const uint32_t at = e & 2047u;
          const uint32_t len = j < n_jobs ? ((e >> 11) & 31u) + 1u : 0u;
          const uint32_t base = place_of(e);
          const uint32_t* word = text + (at >> 2);
          const uint32_t shift = 8u * (at & 3u);
          uint32_t w0 = word[0], w1 = word[1];
#pragma unroll 1
          for (uint32_t o = 0; __ballot(o < len) != 0; o += 8) {           // uniform; eight pairs' values in flight
            if (o < len) {
              const uint32_t w2 = word[(o >> 2) + 2], w3 = word[(o >> 2) + 3];
              const uint32_t bytes[3] = {__builtin_amdgcn_alignbit(w1, w0, shift), __builtin_amdgcn_alignbit(w2, w1, shift),
                                         __builtin_amdgcn_alignbit(w3, w2, shift)};
              w0 = w2;
              w1 = w3;
              uint32_t v[8];
#pragma unroll
              for (int c = 0; c < 8; ++c) {
                // byte-pair table: first byte * 256 + second byte
                const uint32_t pair = (c & 3) == 3 ? __builtin_amdgcn_alignbit(bytes[(c >> 2) + 1], bytes[c >> 2], 24u)
                                                   : bytes[c >> 2] >> (8 * (c & 3));
                const uint32_t swapped = __builtin_amdgcn_perm(0u, pair, 0x0C0C0001u);
                v[c] = kLaneNoPair;
                if (o + c + 1u < len) v[c] = tab.byte_pair[swapped];
              }
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const uint32_t at4 = o + 4 * h;
                if (at4 < len) {
                  *(uint4*)(V + base + at4) = make_uint4(lane_value(v[4 * h], at4), lane_value(v[4 * h + 1], at4 + 1u),
                                                         lane_value(v[4 * h + 2], at4 + 2u), lane_value(v[4 * h + 3], at4 + 3u));
                }
              }
            }
          }
        }
        wave_order();
      }
      {
        // ---- merge: Algorithm 1 on one segment per lane ----
        // The look-ups of the two pairs a merge creates stay in flight over the loop's edge: the next trip first scans
        // the pair values that did not change and only then takes the two new ones.
        // A wave issues one instruction at a time, and what bounds a trip -- of a lone wave too -- is their number, the
        // scalar ones of branches included: so a lane without a segment, or without a look-up, has an address of its own
        // to read and write (kIdle) instead of a branch.
        if (lane < 4) lds[L::kIdle + lane] = kLaneNoPair;
        wave_order();
        uint32_t* const idle_v = lds + L::kIdle;
        uint32_t alive = 0;            // bit o: position o of my segment holds a token; 0: I have no segment
        uint32_t joined = 0;           // bit o: ... one that a merge has made
        uint32_t* v0 = idle_v;         // my segment's first position in V, where its tokens are left as a mask once it is done
        const uint8_t* b0 = (const uint8_t*)text;      // ... and in the text
        uint32_t last = 0;             // where its last four positions begin
        uint32_t next = 0;             // first segment nobody has taken (uniform)
        LaneProbe f1, f2;              // (left token, merged token) and (merged token, token after it)
        f1.q = f2.q = make_uint4(0, 0, 0, 0);
        f1.bucket = f2.bucket = 0;
        f1.tag = f2.tag = kLaneNoTag;
        uint32_t* to1 = idle_v;        // ... where their values go
        uint32_t* to2 = idle_v;
        uint32_t pk = 0, pl = 0;       // ... and their positions
        // A lane without a segment takes the next one of the list.
        auto take_segments = [&]() {
          const uint64_t idle_lanes = __ballot(alive == 0);              // (an idle lane has nothing in flight)
          if (idle_lanes && next < n_jobs) {           // uniform
            const uint32_t mine = next + mbcnt64(idle_lanes);
            next += (uint32_t)__builtin_popcountll(idle_lanes);
            if (alive == 0 && mine < n_jobs) {
              const uint32_t e = jobs[mine];
              const uint32_t top = (e >> 11) & 31u;
              alive = (2u << top) - 1u;
              joined = 0;
              v0 = V + place_of(e);
              b0 = (const uint8_t*)text + (e & 2047u);
              last = top & ~3u;
            }
          }
        };
        take_segments();
        // Every trip ends a segment or removes a token in each lane that has a segment, so so many trips cannot be needed;
        // the bound only guarantees that the loop ends whatever the memory contents.
        const int most_trips = 2 * (int)(upto_part - done) + 64;
        for (int trip = 0; trip < most_trips; ++trip) {
          if (!__ballot(alive != 0)) break;            // every segment is done

          // The lowest value among my pairs, left-most on ties, four positions a load; what is dead or being looked up
          // holds "no pair".  (A lane whose segment does not reach so far reads its last four again.)
          uint32_t best;
          {
            const uint4 a = *(const uint4*)v0, b = *(const uint4*)(v0 + min(4u, last)),
                        c = *(const uint4*)(v0 + min(8u, last)), d = *(const uint4*)(v0 + min(12u, last));
            __builtin_amdgcn_sched_barrier(0);         // (all four loads go out before the first is waited for)
            best = min(min(min(a.x, a.y), min(a.z, a.w)), min(min(b.x, b.y), min(b.z, b.w)));
            best = min(best, min(min(min(c.x, c.y), min(c.z, c.w)), min(min(d.x, d.y), min(d.z, d.w))));
          }
          if (__ballot(last >= 16u)) {                 // uniform
            const uint4 a = *(const uint4*)(v0 + min(16u, last)), b = *(const uint4*)(v0 + min(20u, last)),
                        c = *(const uint4*)(v0 + min(24u, last)), d = *(const uint4*)(v0 + min(28u, last));
            __builtin_amdgcn_sched_barrier(0);         // (likewise)
            best = min(best, min(min(min(a.x, a.y), min(a.z, a.w)), min(min(b.x, b.y), min(b.z, b.w))));
            best = min(best, min(min(min(c.x, c.y), min(c.z, c.w)), min(min(d.x, d.y), min(d.z, d.w))));
          }
          // From here to the issue of the new look-ups a wave is on its way to its next memory round trip: it goes
          // before the waves that are scanning or loading (measured: 1 % on the large workloads).
          __builtin_amdgcn_s_setprio(2);
          {                                            // the two pairs my last merge created
            uint32_t r1, r2;
            lane_probe_finish(tab, f1, f2, r1, r2);
            r1 = lane_value(r1, pl);
            r2 = lane_value(r2, pk);
            *to1 = r1;                                 // (no left neighbour: the same place, to be overwritten)
            *to2 = r2;
            best = min(best, min(r1, r2));
          }
          uint32_t x1 = 0, x2 = 0, y2 = 0;             // (a word without capabilities: no look-up)
          to1 = to2 = idle_v;
          if (best < kLaneInvalid) {                   // (an idle lane has no pair)
            pk = best & 31u;
            const uint32_t upper = alive & (0xFFFFFFFEu << pk);          // not empty: the pair has a right token
            const uint32_t right = (uint32_t)__builtin_ctz(upper);
            const uint32_t after = upper & (upper - 1u);                 // live positions beyond the right token
            const uint32_t lower = alive & ((1u << pk) - 1u);
            pl = lower ? 31u - (uint32_t)__builtin_clz(lower) : pk;
            to2 = v0 + pk;
            to1 = v0 + pl;
            const uint32_t next_at = after ? (uint32_t)__builtin_ctz(after) : 0u;
            const uint32_t next_word = v0[next_at + 1u], next_byte = b0[next_at];
            const uint32_t left_word = to1[1], left_byte = b0[pl];
            y2 = (joined >> next_at) & 1u ? next_word : lane_byte_word(next_byte);
            x1 = (joined >> pl) & 1u ? left_word : lane_byte_word(left_byte);
            y2 = after ? y2 : 0u;
            x1 = lower ? x1 : 0u;
            x2 = lane_merged_word(best);
            *to2 = kLaneNoPair;
            *to1 = kLaneNoPair;
            v0[right] = kLaneNoPair;
            to2[1] = x2;                               // (that position is dead, or has just died)
            alive &= ~(1u << right);
            joined |= 1u << pk;
          } else if (alive != 0) {                     // no pair left: my segment is finished
            *v0 = alive;
            alive = 0;
            last = 0;
            v0 = idle_v;
          }
          lane_probe_start(tab, x1, x2, f1);
          lane_probe_start(tab, x2, y2, f2);
          take_segments();                             // lanes whose segment just ended go on at once
          __builtin_amdgcn_s_setprio(0);
        }
        wave_order();
      }

      // ---- emit: the tokens before a position are its place in the output ----
#pragma unroll 1
      for (uint32_t j0 = 0; j0 < n_jobs; j0 += 64) {   // uniform
        if (j0 + (uint32_t)lane < n_jobs) {
          const uint32_t e = jobs[j0 + (uint32_t)lane];
          const uint32_t at = e & 2047u;
          const uint64_t its_tokens = (uint64_t)V[place_of(e)] << (at & 31u);
          atomicOr(&tokens[at >> 5], (uint32_t)its_tokens);
          if (its_tokens >> 32) atomicOr(&tokens[(at >> 5) + 1u], (uint32_t)(its_tokens >> 32));
        }
      }
      count_tokens();                                  // (of what comes after this part: not yet all)
      if (upto_part == all_places) write_words();      // uniform
      // In the jobs' order, in which neighbours have about as many tokens.  (In the text's order, a store instruction per
      // token of the longest of 64 segments, few lanes in each, was a fifth of the kernel.)
#pragma unroll 1
      for (uint32_t j0 = 0; j0 < n_jobs; j0 += 64) {   // uniform
        uint32_t mine = 0, o = 0, made = 0;
        const uint32_t* v = V;
        const uint8_t* bytes = (const uint8_t*)text;
        if (j0 + (uint32_t)lane < n_jobs) {
          const uint32_t e = jobs[j0 + (uint32_t)lane];
          v = V + place_of(e);
          bytes += e & 2047u;
          mine = v[0];
          o = rank_of(e & 2047u);
          if constexpr (GROUPS)
            if (left) o += lack_of(e & 2047u);         // (left: uniform)
          made = (~mine >> 1) & ((1u << ((e >> 11) & 31u)) - 1u);        // (the position after is of the segment, and dead)
        }
        while (__ballot(mine != 0)) {
          if (mine) {
            const uint32_t q = (uint32_t)__builtin_ctz(mine);
            const uint32_t word = v[q + 1u], byte = bytes[q];
            dst[o++] = (int32_t)((made >> q) & 1u ? word & kTokIdMask : byte);
          }
          mine &= mine - 1u;
        }
      }
      done = upto_part;
    }
    wave_order();                                      // the list's LDS is used again
  }
  // ---- the single bytes, where they are many ----
#pragma unroll 1
  for (uint64_t words = __ballot(singles != 0); words;) {                // uniform: a row of 64 positions at a time
    const int row = (int)__builtin_ctzll(words) >> 1;
    words &= ~(3ull << (2 * row));
    auto row_of = [&](uint32_t word) {
      return (uint32_t)__builtin_amdgcn_readlane((int)word, 2 * row) |
             (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)word, 2 * row + 1) << 32;
    };
    const uint64_t row_tokens = row_of(my_tokens);
    uint32_t o = __builtin_amdgcn_mbcnt_hi((uint32_t)(row_tokens >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)row_tokens,
                                                                     (uint32_t)__builtin_amdgcn_readlane((int)my_rank, 2 * row)));
    if (__builtin_amdgcn_inverse_ballot_w64(row_of(singles))) {
      const uint32_t at = 64u * (uint32_t)row + (uint32_t)lane;
      uint32_t id = ((const uint8_t*)text)[at];
      if constexpr (SPECIAL) {
        if (any_marked) {                              // uniform
          const uint32_t mark = p.cover[begin + at];
          if (mark) id = p.special_base + (mark & kCoverIndex);
        }
      }
      if constexpr (GROUPS)
        if (left) o += lack_of(at);
      dst[o] = (int32_t)id;
    }
  }
  if constexpr (GROUPS) {
    // (empty strings at the end, and lanes without one: nothing after them)
    const uint32_t tokens_before = from < n ? rank_of((uint32_t)from) : total;
    const uint32_t after = lane_read(tokens_before, min(lane + 1, 63));
    if (lane < members) {
      p.counts[s + lane] = (int32_t)((lane + 1 < members ? after : total) - tokens_before);
      if (p.group_ids && !left) p.group_ids[s + lane] = lane == 0 ? (int32_t)total : 0;
    }
  } else {
    if (lane == 63) p.counts[s] = (int32_t)total;
  }
  wave_order();
  return left;
}

// Persistent workgroups, whose waves go over the items of tier 0 on their own.  INLINE: there is no work list, item i is
// string i, and one with a segment that no lane can take goes to the wave-per-item encoder in this kernel.  Else the items
// are groups of strings, or of pieces of strings (see group_members); those of a group that hold such a segment go to
// p.fallback_list, for the kernel that comes after this one, and the group's descriptor is marked for the packing kernel.
// SLOTS: the items are the slots of a small split batch; each wave takes one and finds its piece.
template <class L, bool SPECIAL, bool INLINE, bool SLOTS>
__global__ __launch_bounds__(64 * L::kWaves) void encode_lanes_kernel(EncodeParams p) {
  constexpr bool GROUPS = !INLINE && !SLOTS;
  extern __shared__ __align__(16) uint32_t smem[];
  const uint32_t first = p.list_desc ? p.tier_base[0] : 0u;
  const uint32_t count = p.list_desc ? p.tier_base[1] - first : p.direct_count;
  // The waves that take part: as many as make the rounds even.  5,120 items on 4,096 resident waves
  // are two rounds of 2,560 -- the same two item times, with fewer waves sharing each SIMD.
  const uint32_t n_waves = gridDim.x * L::kWaves;
  const uint32_t rounds = (count + n_waves - 1) / n_waves;
  const uint32_t g = rounds ? (count + rounds - 1) / rounds : 1u;
  // Items per claim: as many as keep every wave of the grid busy, kLaneChunk at most.
  // (Two or three rounds are dealt out whole: with count / g, which is one less unless g divides the count, all
  // waves come back for a claim at the same moment -- 20,011 strings in some 6,000 groups, 50 us or 110.  Each
  // wave's items are neighbours in a list sorted by length, so the first ones get only long items; it is never
  // slower for that: 5,000 pieces of 890 bytes and 5,000 strings of 20 bytes 134 us before, 103 so; 4,500 of each 102,
  // 101; 6,000 of each 110, 110.)
  const uint32_t per_claim = rounds < kLaneChunk ? max(1u, rounds)
                                                 : min(count / g >= 32u ? 2u * kLaneChunk : kLaneChunk, count / g);
  // Neighbouring numbers are waves of different workgroups: few items are spread over the whole chip.
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t b = wave * gridDim.x + blockIdx.x;
  if (blockIdx.x >= g || (uint64_t)blockIdx.x * per_claim >= count) return;   // uniform: nothing for this workgroup
  // Items are claimed kLaneChunk at a time: the first chunk of a wave is its own index, later ones come from
  // the tier's queue head (which starts at zero).  One claim per item would make every wave wait for a round trip
  // to the one contended address after each item.  Lane i fetches the descriptor of the chunk's i-th item, so a
  // chunk costs one round trip for its claim and one for its descriptors.  (Claiming ahead does not pay: loads
  // return in order, so whatever is loaded after the claim waits for it.)
  const int lane = (int)threadIdx.x & 63;
  const ItemDesc* const descs = (const ItemDesc*)p.list_desc;
  auto load_chunk = [&](uint64_t first_item, uint32_t n_items, ItemDesc& d) {
    d.begin = 0;
    d.len = 0;
    d.item = 0;
    const uint64_t item = first_item + (uint32_t)lane;
    if ((uint32_t)lane < n_items) {
      if (descs) {
        d = descs[first + item];
      } else {                                         // no work list: item i is string i
        d.begin = p.offsets[item];
        d.len = (int32_t)(p.offsets[item + 1] - d.begin);
        d.item = (int32_t)item;
      }
    }
  };
  // A wave's own first chunk: per_claim items, and when the list is long zero to three more, by its number,
  // so that the waves do not all come back for their first claim at the same moment (claims on one address
  // are served one after the other, some ten nanoseconds each).
  const uint32_t spread = per_claim >= kLaneChunk ? 1u : 0u;
  constexpr uint32_t kBefore[4] = {0, 0, 1, 3};        // extra items of the waves before b within its group of four
  uint64_t first_item = (uint64_t)b * per_claim + spread * ((b >> 2) * 6u + kBefore[b & 3u]);
  const uint64_t own_items = (uint64_t)g * per_claim + spread * ((g >> 2) * 6u + kBefore[g & 3u]);
  uint32_t here = (uint32_t)min((uint64_t)(per_claim + spread * (b & 3u)), count - min(first_item, (uint64_t)count));
  ItemDesc cur;
  // (on their way while the workgroup's LDS is filled)
  SlotString string{0, 0, 0};
  if constexpr (SLOTS) {
    if (b < g) string = slot_string_of(p.offsets, p.batch, p.piece_target, b);
  } else {
    if (b < g) load_chunk(first_item, here, cur);
  }
  for (int i = (int)threadIdx.x; i < 2048 / 4; i += 64 * L::kWaves)
    ((uint4*)(smem + LaneShared::kCuts))[i] = ((const uint4*)p.table.cuts)[i];
  if (threadIdx.x < 64) {                              // word w of the first l bytes
    const int bytes = (int)(threadIdx.x >> 2) - 4 * (int)(threadIdx.x & 3u);
    smem[LaneShared::kMasks + threadIdx.x] = bytes >= 4 ? 0xFFFFFFFFu : bytes > 0 ? (1u << (8 * bytes)) - 1u : 0u;
  }
  __syncthreads();
  if (b >= g || first_item >= count) return;           // uniform in the wave; no barrier follows
  uint32_t* const arrays = smem + LaneShared::kWords + wave * L::kWords;

  if constexpr (SLOTS) {                               // (the grid covers the slots)
    const SlotPiece piece = slot_piece(p.bytes, string, p.cover, smem + LaneShared::kCuts, p.piece_target, p.max_string, b,
                                       p.slot_string, p.slot_begin, p.slot_len);
    int kind = kSlotDone;
    const int tier = piece.len <= kMemberBytes ? 0 : piece.len <= 4096 ? 1 : piece.len <= 16384 ? 2 : 3;
    if (piece.len < 0 || tier >= p.n_tiers) {          // void, or longer than the host said: nobody encodes it
      if (lane == 0) p.counts[b] = 0;
    } else if (tier > 0) {
      kind = kSlotLeft;
    } else if (encode_item_lanes<L, SPECIAL, false, false>(p, (int)b, piece.begin, piece.len, 1, arrays, smem)) {
      kind = kSlotLeft;
    }
    if (lane == 0) p.slot_kind[b] = kind;
    return;
  }
  auto encode_chunk = [&](uint64_t at, uint32_t here, const ItemDesc& cur) __attribute__((always_inline)) {
    for (uint32_t i = 0; i < here; ++i) {
      const int s = __builtin_amdgcn_readlane(cur.item, (int)i);
      const int n = __builtin_amdgcn_readlane(cur.len, (int)i);
      const int64_t begin = ((int64_t)__builtin_amdgcn_readlane((int)(cur.begin >> 32), (int)i) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)cur.begin, (int)i);
      const int members = GROUPS ? (n >> kGroupShift) & kGroupMask : 1;
      const uint64_t left =
          encode_item_lanes<L, SPECIAL, GROUPS, INLINE>(p, s, begin, GROUPS ? n & kGroupLen : n, members, arrays, smem);
      if (left) {                                      // uniform
        if constexpr (INLINE) {
          wave_order();
          // (the other encoder's arrays take the place of this one's; the bytes' words come from memory, beside their pairs)
          const BlockShared<1> sh = block_shared<1>(arrays + 3 * 1024, p.table.byte_word);
          int64_t its_begin;                           // (read again: kept, they cost registers where few strings come here)
          int its_n;
          item_of(p, s, its_begin, its_n);
          encode_string_segmented<1, 16, true, SPECIAL, false>(p, s, its_begin, its_n, arrays, arrays + 1024, arrays + 2 * 1024,
                                                               sh, Fold{}, nullptr);
          wave_order();
        } else {
          const uint32_t slot = uniform(
              atomicAdd(p.fallback_count, lane == 0 ? (uint32_t)__builtin_popcountll(left) : 0u));
          if ((left >> lane) & 1ull) p.fallback_list[slot + mbcnt64(left)] = s + lane;
          if (lane == 0) ((ItemDesc*)p.list_desc)[first + at + i].len = n | kGroupApart;
        }
      }
      if constexpr (INLINE) {
        // The only string of its batch: this wave finishes the output, for which there is no other launch.
        if (p.out_offsets) {                           // uniform
          __threadfence();                             // (it reads what it has just written)
          const int k = __hip_atomic_load(p.counts + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const int32_t* const ids = left ? p.tmp_ids + begin : p.out_ids;
          if (left || p.id_map)
            for (int o = lane; o < k; o += 64) {
              const int32_t id = __hip_atomic_load(ids + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              p.out_ids[o] = vocabulary_id(p.id_map, id);
            }
          if (lane < 2) p.out_offsets[lane] = lane == 0 ? 0 : k;
        }
      }
    }
  };
  for (;;) {
    encode_chunk(first_item, here, cur);
    if constexpr (INLINE) break;                       // (the grid covers the strings, a wave each)
    if (own_items >= count) break;                     // uniform: the grid's own chunks cover the list
    first_item = own_items + (uint64_t)wave_claim(p.queue_head) * per_claim;
    if (first_item >= count) break;                    // uniform
    here = (uint32_t)min((uint64_t)per_claim, count - first_item);
    load_chunk(first_item, here, cur);
  }
}

}  // namespace bpe
