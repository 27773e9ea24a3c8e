// csrc/word_table.h on the CPU, for tests/test_word_table.py.
#include <cstdint>
#include <map>
#include <utility>

#include "word_table.h"

// Rank of a pair in a table image, as the library asks for it; -1: it is no row.
extern "C" int64_t rank_in_image(const uint32_t* image, int log2_buckets, uint32_t a, uint32_t b) {
  const uint32_t rank = bpe::image_rank(image, log2_buckets, a, b);
  return rank == bpe::kNoRank ? -1 : (int64_t)rank;
}

// Builds the word table of a merge list, with ranks from its table image (as the library does) or, without one, from a map.
// known[t]: the table holds token t.  buckets: capacity words; returns log2 of the number of buckets, or -1 if they do not fit.
extern "C" int build_words(const int32_t* merges, int32_t n, const uint32_t* table_image, int log2_buckets, uint8_t* known,
                           uint32_t* buckets, int64_t capacity, uint32_t* keys) {
  std::map<std::pair<uint32_t, uint32_t>, uint32_t> rank;
  for (int32_t r = 0; r < n; ++r) rank[{(uint32_t)merges[2 * r], (uint32_t)merges[2 * r + 1]}] = (uint32_t)r;
  const auto rank_of = [&](uint32_t a, uint32_t b) {
    if (table_image) return bpe::image_rank(table_image, log2_buckets, a, b);
    const auto it = rank.find({a, b});
    return it == rank.end() ? bpe::kNoRank : it->second;
  };
  bpe::WordImage image;
  bpe::build_words(merges, n, rank_of, image);
  if ((int64_t)image.buckets.size() > capacity) return -1;
  for (size_t i = 0; i < image.buckets.size(); ++i) buckets[i] = image.buckets[i];
  for (size_t i = 0; i < image.keys.size(); ++i) keys[i] = image.keys[i];
  for (size_t t = 0; t < 256 + (size_t)n; ++t) known[t] = t < 256 || image.keys[4 * t + 3] != 0;
  return image.log2_buckets;
}

// The token of `len` bytes as a kernel looks it up, or -1.
extern "C" int32_t find_word(const uint32_t* buckets, int log2_buckets, const uint32_t* keys, const uint8_t* bytes, int len) {
  uint32_t k[4] = {0, 0, 0, (uint32_t)len << 24};
  for (int i = 0; i < len; ++i) k[i >> 2] |= (uint32_t)bytes[i] << (8 * (i & 3));
  const uint32_t hash = bpe::word_hash(k[0], k[1], k[2], k[3]), tag = bpe::word_tag(hash);
  const uint32_t* const bucket = buckets + (size_t)bpe::word_bucket(hash, log2_buckets) * bpe::kWordSlots;
  uint32_t id = bpe::kWordNone;
  for (int i = 0; i < bpe::kWordSlots; ++i) id = (bucket[i] ^ tag) < id ? bucket[i] ^ tag : id;
  if (id >= (1u << bpe::kWordIdBits) - 1u) return -1;
  for (int i = 0; i < 4; ++i)
    if (keys[4 * (size_t)id + i] != k[i]) return -1;
  return (int32_t)id;
}
