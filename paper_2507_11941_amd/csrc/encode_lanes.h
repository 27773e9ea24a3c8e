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
//            where they are cut, and leaves the segments' first positions as a bitmap, then as a list.
//   words    segment-parallel, 64 at a time and four such batches in flight: the segment's bytes are its key; two
//            dependent table reads say which token it is, if it is one.
//   list     the other segments, sorted by length, longest first: a counting sort with one LDS counter per length.
//            Handing the long segments out first is what keeps the lanes level at the end.  Only these segments get a
//            place in the arrays of tokens and pair values (the "arena"), in the list's order.
//   merge    segment-parallel, as above; a lane keeps its segment's liveness as a 32-bit mask, so a segment
//            may have at most 32 bytes.  A string with a longer segment is not encoded here: the kernel hands
//            it to the wave-per-item encoder of encode_segmented.h, which has no such limit.  (An item is one
//            string, a piece of one, or a group of short ones; of a group only such strings are handed on.)
//   emit     segment-parallel: a prefix sum of the segments' token counts gives every one its place in the output
//            (section 4.3's compaction).
//
// words to emit run over as many segments at a time as the arena and the lists hold: in text, all of the item's.
//
// What bounds it is instruction issue: some 2,080 vector and 550 scalar instructions per KiB of text, of which the merge
// loop is two fifths, on four waves a SIMD.  With every segment going through the merges, one item of 1 KiB a wave
// (14.9 trips of the loop per KiB instead of 6.3), the 65,536 documents of the throughput workload took 1,480 us in this
// kernel; they take 985, and the whole call 1,075 instead of 1,659.
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

// What becomes of a segment: its token's number, or one of these.
constexpr uint32_t kRecJob = 1u << 30;          // | its place among the jobs in the text's order
constexpr uint32_t kRecNone = 1u << 31;         // no token

// LDS of a workgroup, in 32-bit words: read-only, shared by its waves.
struct LaneShared {
  static constexpr int kCuts = 0;                                       // bit a + 256 b: bytes a, b have a cut between them
  static constexpr int kByteWord = kCuts + 2048;                        // token word of every byte
  static constexpr int kMasks = kByteWord + 256;                        // [16][4] first l bytes of a key
  static constexpr int kWords = kMasks + 64;
};
// Shape of a workgroup, and the LDS of one of its waves.  WAVES: they take items of their own; BYTES: an item's capacity;
// LIST: segments listed at a time; JOBS: those of them that need merges; ARENA: the bytes of those, in fours.  What bounds
// the number of waves is LDS, and what bounds the kernel is how many waves there are to wait at once: 65,536 documents take
// 1,554 us with 8 waves a CU, 1,379 with 10, 1,232 with 12 (that was with the tokens in a second array beside V) and 1,107
// with the 16 that one array leaves room for.  Twice as long an item takes less than half as many trips of the merge loop
// for each of its bytes (5.4 instead of 12.2 per KiB: the longest chain of merges is 10 long in either): the same batch in
// items of 1 KiB took 1,443 instead of 1,232.  A small batch wants each piece of text to have a wave.
template <int BYTES, int WAVES, int LIST, int JOBS, int ARENA, int AT_LEAST>
struct LaneShape {
  static constexpr int kBytes = BYTES, kWaves = WAVES, kListed = LIST, kMostJobs = JOBS, kArena = ARENA;
  static constexpr int kText = 0;                                       // the item's bytes; a key's words reach beyond them
  static constexpr int kStrings = kText + BYTES / 4 + 8;                // (groups) bit p: a string starts at p
  static constexpr int kList = kStrings + BYTES / 32;                   // uint16 first position of a segment
  static constexpr int kJobs = kList + LIST / 2 + 2;                    // the jobs sorted: first position | (length - 1) << 11 |
                                                                        //   place << 16, then arena position / 4 << 16 instead
  static constexpr int kPlaces = kJobs + JOBS;                          // uint16 arena position of the jobs in the text's order
  static constexpr int kHist = kPlaces + JOBS / 2;                      // jobs of each length, then list bases
  static constexpr int kV = (kHist + 32 + 3) / 4 * 4;                   // a word for every arena position
  static constexpr int kIdle = kV + ARENA;                              // what a lane without a segment reads and writes
  static constexpr int kEnd = kIdle + 4;
  // before the arena is used:
  static constexpr int kStarts = kV;                                    // bit p: a segment starts at p, or the item ends
  static constexpr int kFirstJobs = kV;                                 // the jobs in the text's order
  static constexpr int kFound = kV + JOBS;                              // what becomes of a segment
  static constexpr int kWords = ((kEnd > AT_LEAST ? kEnd : AT_LEAST) + 3) / 4 * 4;
  static constexpr size_t kLdsBytes = lds_blocks(sizeof(uint32_t) * (LaneShared::kWords + WAVES * kWords));
  static_assert(kText % 4 == 0 && ARENA % 4 == 0, "wide loads and stores");
  static_assert(ARENA <= 2048 && BYTES <= 2048 && BYTES % 1024 == 0 && LIST % 64 == 0 && LIST <= 512 && JOBS % 64 == 0,
                "fields of the packed words; a lane per word of the bitmap");
  static_assert(JOBS + LIST <= ARENA && BYTES / 32 + 4 <= ARENA, "what shares a place fits it");
  static_assert(kLdsBytes <= 160 * 1024, "one workgroup a CU");
};
using LargeItems = LaneShape<kGroupBytes, 16, 448, 256, 1152, 0>;
using SmallItems = LaneShape<kMemberBytes, 16, 256, 128, 704, 0>;
// (the arrays of the one-wave encoder that takes a string over)
constexpr int kOtherWords = encode_array_words<1, 16, false, true>() + encode_exchange_words<1>();
using InlineItems = LaneShape<kMemberBytes, 12, 256, 128, 704, kOtherWords>;

__device__ inline uint32_t mbcnt64(uint64_t mask) {                     // set bits of mask below my lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
// Where a segment that is done keeps its place in the output, its tokens being the mask in its first word: at its second
// token, whose pair no longer counts, or behind the one token's word (a segment has four words at least).
__device__ inline uint32_t lane_spare(uint32_t tokens) {
  return tokens & (tokens - 1u) ? (uint32_t)__builtin_ctz(tokens & (tokens - 1u)) : 2u;
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

// Bytes at ... at + 15 of the `room` bytes from src on, whatever their alignment; 0 <= at < room, and what lies beyond
// them reads as anything.  `before`: bytes that may be read before src as well.
__device__ inline uint4 load_16_bytes(const uint8_t* src, int at, int64_t before, int64_t room) {
  uint4 v = make_uint4(0, 0, 0, 0);
  const int last = (int)min(room, (int64_t)1 << 30) - 16;                // (uniform)
  if (before + last < 0) {                             // uniform: fewer than 16 bytes in all
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int j = 0; j < (int)room; ++j) {
      const uint32_t b = src[j];
      const int to = j - at;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (to >> 2 == i) w[i] |= b << (8 * (to & 3));
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
  const int from = min(at, last);
  __builtin_memcpy(&v, src + (int64_t)from, 16);
  const uint32_t skip = (uint32_t)(at - from);         // 0 but at the end
  if (__ballot(skip != 0)) {
    if (skip & 8u) { v.x = v.z; v.y = v.w; }
    if (skip & 4u) { v.x = v.y; v.y = v.z; v.z = v.w; }
    const uint32_t bits = 8u * (skip & 3u);
    v.x = __builtin_amdgcn_alignbit(v.y, v.x, bits);
    v.y = __builtin_amdgcn_alignbit(v.z, v.y, bits);
    v.z = __builtin_amdgcn_alignbit(v.w, v.z, bits);
    v.w >>= bits;
  }
  return v;
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
  uint16_t* const list = (uint16_t*)(lds + L::kList);
  uint32_t* const jobs = lds + L::kJobs;
  uint16_t* const places = (uint16_t*)(lds + L::kPlaces);
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
          uint32_t marked = 0;
          if (__ballot((m.x | m.y | m.z | m.w) != 0)) {
            any_marked = true;
            const uint32_t mw[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
            for (int j = 0; j < 16; ++j) marked |= (((mw[j >> 2] >> (8 * (j & 3))) & 0xFFu) ? 1u : 0u) << j;
            if (at < n && n - at < 16) marked &= (1u << (n - at)) - 1u;      // (the next string's, or none)
          }
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
  uint32_t my_starts = lane < n_words ? starts[lane] : 0u;
  {
    const uint32_t next = lane < n_words ? starts[lane + 1] : 0u;
    const int top = 32 * lane + 31 - (int)__builtin_clz(my_starts | 1u);   // the word's last start
    const bool empty = lane < n_words && my_starts == 0;
    const bool gap = my_starts != 0 && next != 0 && top < n &&
                     __builtin_clz(my_starts) + __builtin_ctz(next | 0x80000000u) + 1 > kLaneSegmentMax;
    uint64_t too_long = __ballot(empty || gap);
    if (too_long) {                                    // uniform
      if constexpr (!GROUPS) return 1;
      // The strings that hold one: lane m asks for string m.  Of their segments only the first start is kept; so long a
      // one gets no token below.
      const int inside = empty ? 32 * lane : top;
      for (; too_long; too_long &= too_long - 1ull) {  // uniform
        const int at = __builtin_amdgcn_readlane(inside, (int)__builtin_ctzll(too_long));
        left |= __ballot(from <= at && at < to);
      }
      for (uint64_t m = left; m; m &= m - 1ull) {      // uniform
        const int lo = max(__builtin_amdgcn_readlane(from, (int)__builtin_ctzll(m)) + 1 - 32 * lane, 0);
        const int hi = min(__builtin_amdgcn_readlane(to, (int)__builtin_ctzll(m)) - 32 * lane, 32);
        if (lo < hi) my_starts &= ~((hi >= 32 ? 0xFFFFFFFFu : (1u << hi) - 1u) & (0xFFFFFFFFu << lo));
      }
    }
  }
  if (32 * lane + 31 >= n && lane < n_words && (n & 31)) my_starts &= (1u << (n & 31)) - 1u;   // the end is no start
  const uint32_t my_count = (uint32_t)__builtin_popcount(my_starts);
  const uint32_t starts_upto = wave_scan<OpAdd>(my_count, 0u);

  int32_t* const dst = ALONE && p.out_offsets ? p.out_ids : p.tmp_ids + begin;
  // Single bytes all (blank lines, padding that no row joins): their ids are the bytes.  (64 strings of 64 KiB of spaces: 16 us,
  // as segments 48.)
  if ((int)__builtin_amdgcn_readlane((int)starts_upto, 63) == n && !any_marked) {        // uniform
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
  uint32_t total = 0;                                  // tokens of the segments done (uniform)
  uint32_t tokens_before = 0;                          // (groups) of string `lane`
  uint32_t lack = 0;                                   // (apart) what the place of a token lacks to its string's own
  uint32_t listed_before = 0;                          // segments of earlier lists (uniform)
  uint32_t my_segment = 0xFFFFFFFFu;                   // (groups) the one that string `lane` starts with
  if constexpr (GROUPS) {
    const int word = min(from >> 5, 63);
    const uint32_t before = lane_read(starts_upto - my_count, word);
    const uint32_t bits = lane_read(my_starts, word);
    if (from < n) my_segment = before + (uint32_t)__builtin_popcount(bits & ((1u << (from & 31)) - 1u));
  }
  for (int word0 = 0; word0 < n_words;) {              // (a list of the whole item, unless it has very many segments)
    // ---- list of the segments that start in words word0 ... word1 - 1 ----
    const uint64_t in_list = __ballot(lane >= word0 && lane < n_words && starts_upto - listed_before <= (uint32_t)L::kListed);
    const int word1 = word0 + (int)__builtin_popcountll(in_list);          // (at least one more: a word has 32 starts)
    const uint32_t listed_upto = (uint32_t)__builtin_amdgcn_readlane((int)starts_upto, word1 - 1);
    const int n_listed = (int)(listed_upto - listed_before);
    {
      const uint64_t later = __ballot(lane >= word1 && my_starts != 0);
      const int first = 32 * lane + (int)__builtin_ctz(my_starts | 0x80000000u);
      const int end = later ? __builtin_amdgcn_readlane(first, (int)__builtin_ctzll(later)) : n;
      uint32_t at = starts_upto - my_count - listed_before;
      uint32_t m = lane >= word0 && lane < word1 ? my_starts : 0u;
      while (__ballot(m != 0)) {
        if (m) list[at++] = (uint16_t)(32 * lane + (int)__builtin_ctz(m));
        m &= m - 1u;
      }
      if (lane == 0) list[n_listed] = (uint16_t)end;
    }
    wave_order();
    word0 = word1;
    const uint32_t list_first = listed_before;
    listed_before = listed_upto;

    for (int i0 = 0; i0 < n_listed;) {                 // uniform
      // ---- words: which segments are one token ----
      int i1 = i0;                                     // segments from i0 to here are done in this round
      uint32_t n_jobs = 0, used = 0;                   // those that need merges, and their places in the arena (uniform)
      const int round_end = min(n_listed, i0 + L::kListed);
      bool full = false;                               // uniform
      while (i1 < round_end && !full) {                // uniform
        uint32_t k[kLaneBatches][4], first[kLaneBatches], len[kLaneBatches], mark[kLaneBatches], tag[kLaneBatches];
        uint4 bucket[kLaneBatches], key[kLaneBatches];
        const int base = i1;
#pragma unroll
        for (int r = 0; r < kLaneBatches; ++r) {
          const int i = min(base + 64 * r + lane, n_listed - 1);
          first[r] = list[i];
          len[r] = (uint32_t)list[i + 1] - first[r];
        }
#pragma unroll
        for (int r = 0; r < kLaneBatches; ++r) {
          if (base + 64 * r + lane >= n_listed) len[r] = 0;
          const uint32_t* const word = text + (first[r] >> 2);
          const uint32_t shift = 8u * (first[r] & 3u);
          const uint4 mask = *(const uint4*)(shared + LaneShared::kMasks + 4 * min(len[r], (uint32_t)kWordBytes));
          k[r][0] = __builtin_amdgcn_alignbit(word[1], word[0], shift) & mask.x;
          k[r][1] = __builtin_amdgcn_alignbit(word[2], word[1], shift) & mask.y;
          k[r][2] = __builtin_amdgcn_alignbit(word[3], word[2], shift) & mask.z;
          k[r][3] = (__builtin_amdgcn_alignbit(word[4], word[3], shift) & mask.w) | (len[r] << 24);
        }
#pragma unroll
        for (int r = 0; r < kLaneBatches; ++r) {
          tag[r] = mark[r] = 0;
          bucket[r] = make_uint4(kWordNone, kWordNone, kWordNone, kWordNone);
          if (__ballot(len[r] > 1u)) {                 // uniform: else single bytes all, or nothing
            const uint32_t hash = word_hash(k[r][0], k[r][1], k[r][2], k[r][3]);
            tag[r] = word_tag(hash);
            if (len[r] - 2u <= (uint32_t)kWordBytes - 2u)
              bucket[r] = tab.word_buckets[word_bucket(hash, tab.log2_word_buckets)];
          }
          if constexpr (SPECIAL)
            if (len[r] == 1u) mark[r] = p.cover[begin + first[r]];
        }
#pragma unroll
        for (int r = 0; r < kLaneBatches; ++r) {
          // (at most one slot of a bucket has the tag; an empty one leaves all ones in the id's bits at best)
          tag[r] = min(min(bucket[r].x ^ tag[r], bucket[r].y ^ tag[r]), min(bucket[r].z ^ tag[r], bucket[r].w ^ tag[r]));
          key[r] = make_uint4(0, 0, 0, 0);
          if (tag[r] < (1u << kWordIdBits) - 1u) key[r] = tab.word_keys[tag[r]];
        }
#pragma unroll
        for (int r = 0; r < kLaneBatches; ++r) {
          if (base + 64 * r < round_end && !full) {    // uniform
            const bool same = len[r] - 2u <= (uint32_t)kWordBytes - 2u &&          // (then no key of zeros is its own)
                              ((key[r].x ^ k[r][0]) | (key[r].y ^ k[r][1]) | (key[r].z ^ k[r][2]) | (key[r].w ^ k[r][3])) == 0;
            uint32_t what = same ? tag[r] : kRecNone;
            const bool job = !same && len[r] - 2u <= (uint32_t)kLaneSegmentMax - 2u;
            if (len[r] == 1u) {
              what = k[r][0];
              if constexpr (SPECIAL)
                if (mark[r]) what = (mark[r] & kCoverFirst) ? p.special_base + (mark[r] & kCoverIndex) : kRecNone;
            }
            int taken = 64;
            const uint64_t job_lanes = __ballot(job);
            if (job_lanes) {                           // uniform
              const uint32_t upto = used + wave_scan<OpAdd>(job ? (len[r] + 3u) & ~3u : 0u, 0u);
              const uint32_t place = n_jobs + mbcnt64(job_lanes);
              const uint64_t misfit = __ballot(job && (upto > (uint32_t)L::kArena || place >= (uint32_t)L::kMostJobs));
              if (misfit) {                            // uniform: the round ends before this segment
                taken = (int)__builtin_ctzll(misfit);
                full = true;
              }
              if (job && lane < taken) {
                lds[L::kFirstJobs + place] = first[r] | ((len[r] - 1u) << 11) | (place << 16);
                what = kRecJob | place;
              }
              n_jobs += (uint32_t)__builtin_popcountll(taken < 64 ? job_lanes & ((1ull << taken) - 1ull) : job_lanes);
              if (taken > 0) used = (uint32_t)__builtin_amdgcn_readlane((int)upto, taken - 1);
            }
            lds[L::kFound + base - i0 + 64 * r + lane] = what;     // (of what is not taken, looked up again)
            i1 = min(base + 64 * r + taken, round_end);
          }
        }
      }
      if (lane < 32) hist[lane] = 0;
      wave_order();
      uint32_t found[L::kListed / 64];                  // what becomes of segment i0 + 64 r + lane
#pragma unroll
      for (int r = 0; r < L::kListed / 64; ++r) found[r] = lds[L::kFound + 64 * r + lane];
      wave_order();

      if (n_jobs) {                                    // uniform
        // ---- list: the segments that need merges, longest first (counting sort over the 31 possible lengths) ----
        constexpr int kRounds = L::kMostJobs / 64;
        uint32_t entry[kRounds], place[kRounds];       // (entry: as in kJobs)
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
          entry[r] = place[r] = 0;
          if (64u * r + (uint32_t)lane < n_jobs) {
            entry[r] = lds[L::kFirstJobs + 64 * r + lane];
            place[r] = atomicAdd(&hist[31u - ((entry[r] >> 11) & 31u)], 1u);   // my place among those of my length
          }
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
        for (int r = 0; r < kRounds; ++r)
          if (64u * r + (uint32_t)lane < n_jobs) jobs[hist[31u - ((entry[r] >> 11) & 31u)] + place[r]] = entry[r];
        wave_order();
        // ---- their places in the arena: byte-level pre-tokenisation (section 4.1) and the initial pair values ----
        uint32_t arena = 0;                            // uniform
#pragma unroll 1
        for (uint32_t j0 = 0; j0 < n_jobs; j0 += 64) { // uniform
          const uint32_t j = j0 + (uint32_t)lane;
          const uint32_t e = jobs[min(j, n_jobs - 1u)];
          const uint32_t at = e & 2047u;
          const uint32_t len = j < n_jobs ? ((e >> 11) & 31u) + 1u : 0u;
          const uint32_t room = (len + 3u) & ~3u;
          const uint32_t upto = arena + wave_scan<OpAdd>(room, 0u);
          const uint32_t base = upto - room;
          arena = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
          wave_order();                                 // (all lanes have read their entries)
          if (len) {
            jobs[j] = (e & 0xFFFFu) | (base << 14);
            places[e >> 16] = (uint16_t)base;
          }
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
      if (n_jobs) {                                    // uniform
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
              v0 = V + 4u * (e >> 16);
              b0 = (const uint8_t*)text + (e & 2047u);
              last = top & ~3u;
            }
          }
        };
        take_segments();
        // Every trip ends a segment or removes a token in each lane that has a segment, so so many trips cannot be needed;
        // the bound only guarantees that the loop ends whatever the memory contents.
        const int most_trips = 2 * (int)used + 64;
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
            for (uint32_t o = 16; o < 32; o += 4) {
              const uint4 a = *(const uint4*)(v0 + min(o, last));
              best = min(best, min(min(a.x, a.y), min(a.z, a.w)));
            }
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

      // ---- emit: a prefix sum of the segments' token counts gives every one its place ----
      // First the segments that are one token, in the text's order; then the others, in the jobs' order: neighbours there
      // have about as many tokens.  (In the text's order too, a store instruction per token of the longest of 64 segments,
      // few lanes in each, was a fifth of the kernel.)
#pragma unroll
      for (int r = 0; r < L::kListed / 64; ++r) {
        const int b = i0 + 64 * r;
        if (b >= i1) continue;                         // uniform
        const int i = b + lane;
        const uint32_t what = i < i1 ? found[r] : kRecNone;
        uint32_t count = what < kRecJob ? 1u : 0u;
        uint32_t at = 0, tokens = 0;
        if (what & kRecJob) {
          at = places[what & (uint32_t)(L::kMostJobs - 1)];
          tokens = V[at];
          count = (uint32_t)__builtin_popcount(tokens);
        }
        const uint32_t upto = total + wave_scan<OpAdd>(count, 0u);
        uint32_t o = upto - count;
        if constexpr (GROUPS) {                        // my string's first segment is one of these: its tokens begin there
          const uint32_t which = my_segment - (list_first + (uint32_t)b);
          const uint32_t its = lane_read(o, (int)(which & 63u));
          if (which < 64u && b + (int)which < i1) tokens_before = its;
          if (left) {                                  // uniform: strings at their own places
            const uint32_t pos = i < i1 ? list[i] : 0u;
            const uint64_t heads = __ballot(i < i1 && ((strings[pos >> 5] >> (pos & 31u)) & 1u));
            const uint64_t upto_me = heads & (~0ull >> (63 - lane));
            const uint32_t mine = pos - o;             // (of a string's first segment)
            const uint32_t its_lack = lane_read(mine, upto_me ? 63 - (int)__builtin_clzll(upto_me) : lane);
            o += upto_me ? its_lack : lack;
            if (heads) lack = (uint32_t)__builtin_amdgcn_readlane((int)mine, 63 - (int)__builtin_clzll(heads));
          }
        }
        if (what < kRecJob) dst[o] = (int32_t)what;
        if (what & kRecJob) V[at + lane_spare(tokens)] = o;
        total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
      }
      wave_order();
#pragma unroll 1
      for (uint32_t j0 = 0; j0 < n_jobs; j0 += 64) {   // uniform
        uint32_t tokens = 0, o = 0, made = 0;
        const uint32_t* v = V;
        const uint8_t* bytes = (const uint8_t*)text;
        if (j0 + (uint32_t)lane < n_jobs) {
          const uint32_t e = jobs[j0 + (uint32_t)lane];
          v = V + 4u * (e >> 16);
          bytes += e & 2047u;
          tokens = v[0];
          o = v[lane_spare(tokens)];
          made = (~tokens >> 1) & ((1u << ((e >> 11) & 31u)) - 1u);      // (the position after is of the segment, and dead)
        }
        while (__ballot(tokens != 0)) {
          if (tokens) {
            const uint32_t q = (uint32_t)__builtin_ctz(tokens);
            const uint32_t word = v[q + 1u], byte = bytes[q];
            dst[o++] = (int32_t)((made >> q) & 1u ? word & kTokIdMask : byte);
          }
          tokens &= tokens - 1u;
        }
      }
      wave_order();                                     // the round's LDS is used again
      i0 = i1;
    }
  }
  if constexpr (GROUPS) {
    if (from >= n) tokens_before = total;              // (empty strings at the end, and lanes without one)
    const uint32_t after = lane_read(tokens_before, min(lane + 1, 63));
    if (lane < members) {
      p.counts[s + lane] = (int32_t)((lane + 1 < members ? after : total) - tokens_before);
      if (p.group_ids && !left) p.group_ids[s + lane] = lane == 0 ? (int32_t)total : 0;
    }
  } else {
    if (lane == 63) p.counts[s] = (int32_t)total;
  }
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
  const uint32_t first = p.list ? p.tier_base[0] : 0u;
  const uint32_t count = p.list ? p.tier_base[1] - first : p.direct_count;
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
  for (int i = (int)threadIdx.x; i < 2048 / 4; i += 64 * L::kWaves)
    ((uint4*)(smem + LaneShared::kCuts))[i] = ((const uint4*)p.table.cuts)[i];
  for (int i = (int)threadIdx.x; i < 256; i += 64 * L::kWaves) smem[LaneShared::kByteWord + i] = p.table.byte_word[i];
  if (threadIdx.x < 64) {                              // word w of the first l bytes
    const int bytes = (int)(threadIdx.x >> 2) - 4 * (int)(threadIdx.x & 3u);
    smem[LaneShared::kMasks + threadIdx.x] = bytes >= 4 ? 0xFFFFFFFFu : bytes > 0 ? (1u << (8 * bytes)) - 1u : 0u;
  }
  __syncthreads();
  if (b >= g || (uint64_t)b * per_claim >= count) return;   // uniform in the wave; no barrier follows
  uint32_t* const arrays = smem + LaneShared::kWords + wave * L::kWords;

  // Items are claimed kLaneChunk at a time: the first chunk of a wave is its own index, later ones come from
  // the tier's queue head (which starts at zero).  One claim per item would make every wave wait for a round trip
  // to the one contended address after each item.  Lane i fetches the descriptor of the chunk's i-th item, so a
  // chunk costs one round trip for its claim and one for its descriptors.  (Claiming ahead does not pay: loads
  // return in order, so whatever is loaded after the claim waits for it.)
  const int lane = (int)threadIdx.x & 63;
  if constexpr (SLOTS) {                               // (the grid covers the slots)
    const SlotPiece piece = slot_piece(p.bytes, p.offsets, p.batch, p.cover, smem + LaneShared::kCuts, p.piece_target,
                                       p.max_string, b, p.slot_string, p.slot_begin, p.slot_len);
    int kind = kSlotDone;
    const int tier = piece.len <= kMemberBytes ? 0 : piece.len <= 4096 ? 1 : piece.len <= 16384 ? 2 : 3;
    if (piece.len < 0 || tier >= p.n_tiers) {          // void, or longer than the host said: nobody encodes it
      if (lane == 0) p.counts[b] = 0;
    } else if (tier > 0) {
      kind = kSlotDone + 1 + tier;
    } else if (encode_item_lanes<L, SPECIAL, false, false>(p, (int)b, piece.begin, piece.len, 1, arrays, smem)) {
      kind = kSlotPassed;
    }
    if (lane == 0) p.slot_kind[b] = kind;
    return;
  }
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
          // (the other encoder's arrays take the place of this one's)
          const BlockShared<1> sh = block_shared<1>(arrays + 3 * 1024, smem + LaneShared::kByteWord);
          encode_string_segmented<1, 16, true, SPECIAL>(p, s, arrays, arrays + 1024, arrays + 2 * 1024, sh);
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
  // A wave's own first chunk: per_claim items, and when the list is long zero to three more, by its number,
  // so that the waves do not all come back for their first claim at the same moment (claims on one address
  // are served one after the other, some ten nanoseconds each).
  const uint32_t spread = per_claim >= kLaneChunk ? 1u : 0u;
  constexpr uint32_t kBefore[4] = {0, 0, 1, 3};        // extra items of the waves before b within its group of four
  uint64_t first_item = (uint64_t)b * per_claim + spread * ((b >> 2) * 6u + kBefore[b & 3u]);
  const uint64_t own_items = (uint64_t)g * per_claim + spread * ((g >> 2) * 6u + kBefore[g & 3u]);
  if (first_item >= count) return;                     // uniform
  uint32_t here = (uint32_t)min((uint64_t)(per_claim + spread * (b & 3u)), count - first_item);
  ItemDesc cur;
  load_chunk(first_item, here, cur);
  for (;;) {
    encode_chunk(first_item, here, cur);
    if (own_items >= count) break;                     // uniform: the grid's own chunks cover the list
    // (lane 0 adds 1; every lane takes part, so that no lane-dependent branch sits at the loop's edge)
    const uint32_t claimed = atomicAdd(p.queue_head, lane == 0 ? 1u : 0u);
    first_item = own_items + (uint64_t)uniform(claimed) * per_claim;
    if (first_item >= count) break;                    // uniform
    here = (uint32_t)min((uint64_t)per_claim, count - first_item);
    load_chunk(first_item, here, cur);
  }
}

}  // namespace bpe
