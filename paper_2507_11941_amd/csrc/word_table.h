// Whole segments that are one token: a second table beside the merge table, from a segment's bytes to its token.
//
// A segment (a stretch between two cuts, see table_format.h) is encoded on its own, so its tokens depend on nothing but
// its bytes; and of a word-like text's segments two in three to five in six ARE one token of the vocabulary, after three
// quarters or more of all merges.  Those are looked up as a whole.  The table holds every token of 2 to kWordBytes bytes
// whose bytes Algorithm 1 turns into just that token; whatever is not found in it goes through the merges.  So it may
// leave tokens out at will: a full bucket takes no more.
//
//   * Key: the bytes, zero-padded to 15, and their number in the 16th: four words, compared in full.
//   * Bucket: four slots of 32 bits, token id | 12 bits of the key's hash << 20, one 16-byte load; no two slots of a
//     bucket have the same 12 bits.  A slot that matches them names the token whose key is then read (16 bytes at
//     keys[id]) and compared, so that there are no false hits.  Tokens go in by rank, the most frequent first; with 2.5
//     slots or more per word, one word in sixty finds its bucket full.
//
// 100,000 rows: 1 MiB of buckets and 1.6 MB of keys (of which a text's frequent words touch a small part).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <new>
#include <vector>

#include "table_format.h"

namespace bpe {

constexpr int kWordBytes = 15;
constexpr int kWordSlots = 4;
constexpr int kWordIdBits = 20;
constexpr uint32_t kWordNone = 0xFFFFFFFFu;      // empty slot
constexpr int kMinLog2WordBuckets = 6;

// k3: bytes 12..14 and the length.
BPE_HD uint32_t word_hash(uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3) {
  const uint64_t p = (uint64_t)(k0 ^ 0xA3F1C28Du) * (k1 ^ 0x6D2E9B57u);
  const uint64_t q = (uint64_t)(k2 ^ 0x94D04BB1u) * (k3 ^ 0x3C6EF372u);
  const uint64_t r = (uint64_t)((uint32_t)p ^ (uint32_t)(q >> 32) ^ 0x5851F42Du) * ((uint32_t)(p >> 32) ^ (uint32_t)q ^ 0xB5297A4Du);
  return (uint32_t)r ^ (uint32_t)(r >> 32);
}
BPE_HD uint32_t word_bucket(uint32_t hash, int log2_buckets) { return hash >> (32 - log2_buckets); }
BPE_HD uint32_t word_tag(uint32_t hash) { return hash << kWordIdBits; }        // the hash's low 12 bits, in a slot's place

// Row of the pair (a, b) in a table image (see table_format.h; its buckets come first), or a value above all rows.
inline uint32_t image_rank(const uint32_t* image, int log2_buckets, uint32_t a, uint32_t b) {
  const Placement pl = place_pair(a, b, log2_buckets);
  const uint32_t* const home = image + (size_t)pl.bucket * kSlotsPerBucket * 2;
  const uint32_t reach = home[3] == 0xFFFFFFFFu ? 0u : bucket_reach(home[0], home[2]);
  for (uint32_t d = 0; d <= reach; ++d) {
    const uint32_t* const bucket = image + (size_t)(pl.bucket ^ d) * kSlotsPerBucket * 2;
    for (int k = 0; k < kSlotsPerBucket; ++k)
      if (bucket[2 * k + 1] == slot_tag(pl.fingerprint, d)) return bucket[2 * k] >> kRankShift;
  }
  return kNoRank;
}

// Does Algorithm 1 turn the bytes of row t's token into that token?  known[x]: the answer for every older token.
// It does if it does so for both operands and no merge joins a token of the left one's bytes with a token of the right
// one's before both are whole.  What stands at the boundary meanwhile are the tokens down the left operand's right edge
// and down the right operand's left edge, smallest first; each stands there until the row that makes the next one, and
// ranks decide which row comes when: rows only use older tokens, so both edges grow in the order of their ranks.
// rank_of(a, b): the row of a pair, or a value above all rows.
template <class RankOf>
inline bool encodes_to_itself(const int32_t* merges, int32_t row, const std::vector<uint8_t>& known, const RankOf& rank_of) {
  const int32_t left = merges[2 * row], right = merges[2 * row + 1];
  if (!known[(size_t)left] || !known[(size_t)right]) return false;
  int32_t l_edge[kWordBytes], r_edge[kWordBytes];      // from the whole operand down to a byte
  int l = 0, r = 0;
  for (l_edge[0] = left; l_edge[l] >= 256; ++l) l_edge[l + 1] = merges[2 * (l_edge[l] - 256) + 1];
  for (r_edge[0] = right; r_edge[r] >= 256; ++r) r_edge[r + 1] = merges[2 * (r_edge[r] - 256)];
  while (l > 0 || r > 0) {
    const uint32_t until_l = l > 0 ? (uint32_t)(l_edge[l - 1] - 256) : 0xFFFFFFFFu;    // the row that ends its stay
    const uint32_t until_r = r > 0 ? (uint32_t)(r_edge[r - 1] - 256) : 0xFFFFFFFFu;
    const uint32_t across = rank_of((uint32_t)l_edge[l], (uint32_t)r_edge[r]);
    // (equal ranks are the same pair: the left-most goes first, so the boundary's goes before the right operand's)
    if (across < until_l && across <= until_r) return false;
    if (until_l <= until_r) --l; else --r;
  }
  return true;
}

// The host's copy of the table.
struct WordImage {
  int log2_buckets = kMinLog2WordBuckets;
  std::vector<uint32_t> buckets;                       // [2^log2_buckets][kWordSlots]
  std::vector<uint32_t> keys;                          // [256 + rows][4], zero for tokens that are not in the table
};
// merges: checked rows in the library's numbering.  Throws std::bad_alloc.
template <class RankOf>
inline void build_words(const int32_t* merges, int32_t n_merges, const RankOf& rank_of, WordImage& out) {
  typedef unsigned __int128 key_t;                     // (its bytes, little-endian, are the key's)
  static_assert(kWordBytes == 15, "a key's last byte is its length");
  const size_t n_tokens = 256 + (size_t)n_merges;
  std::vector<key_t> bytes(n_tokens);                  // ... without the length
  std::vector<uint8_t> length(n_tokens, 0), known(n_tokens, 0);    // length 0: more than kWordBytes
  for (size_t b = 0; b < 256; ++b) {
    length[b] = known[b] = 1;
    bytes[b] = (key_t)b;
  }
  size_t n_words = 0;
  for (int32_t row = 0; row < n_merges; ++row) {
    const size_t left = (size_t)merges[2 * row], right = (size_t)merges[2 * row + 1], t = 256 + (size_t)row;
    if (!length[left] || !length[right] || length[left] + length[right] > kWordBytes) continue;
    length[t] = (uint8_t)(length[left] + length[right]);
    bytes[t] = bytes[left] | bytes[right] << (8 * length[left]);
    known[t] = encodes_to_itself(merges, row, known, rank_of);
    n_words += known[t];
  }
  out.log2_buckets = kMinLog2WordBuckets;
  while (((size_t)kWordSlots << out.log2_buckets) * 2 < n_words * 5) ++out.log2_buckets;
  out.buckets.assign((size_t)kWordSlots << out.log2_buckets, kWordNone);
  out.keys.assign(n_tokens * 4, 0);
  for (size_t t = 256; t < n_tokens; ++t) {
    if (!known[t]) continue;
    const uint32_t k[4] = {(uint32_t)bytes[t], (uint32_t)(bytes[t] >> 32), (uint32_t)(bytes[t] >> 64),
                           (uint32_t)(bytes[t] >> 96) | (uint32_t)length[t] << 24};
    const uint32_t hash = word_hash(k[0], k[1], k[2], k[3]), tag = word_tag(hash);
    uint32_t* const bucket = out.buckets.data() + (size_t)word_bucket(hash, out.log2_buckets) * kWordSlots;
    int place = -1;
    for (int i = 0; i < kWordSlots; ++i) {
      if (bucket[i] == kWordNone) { place = i; break; }
      if ((bucket[i] ^ tag) >> kWordIdBits == 0) break;
    }
    if (place < 0) continue;                           // its segments go through the merges
    bucket[place] = tag | (uint32_t)t;
    for (int i = 0; i < 4; ++i) out.keys[t * 4 + i] = k[i];
  }
}

}  // namespace bpe
