// Batch-level kernels around the per-string encoder: length binning (which kernel variant encodes which
// string, longest strings first), the cutting of long strings into pieces at segment cuts, the marking of
// special-token occurrences, the scan of token counts into out_offsets, and the packing of the per-item id
// runs into the dense output (the paper only says that the result is an id tensor, section 2.2; the dense
// ids + offsets layout is this library's).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "piece_slots.h"
#include "string_groups.h"
#include "table_format.h"

namespace bpe {

constexpr int kMaxTiers = 4;
constexpr int kLenBuckets = 64;                      // length classes inside a tier, longest first
constexpr int kBinKeys = kMaxTiers * kLenBuckets;

struct TierPlan {
  int n_tiers;
  int cap[kMaxTiers];                                // tier t takes strings with cap[t-1] < len <= cap[t]
};

// Control block at the start of the workspace.
struct Control {
  uint32_t tier_base[kMaxTiers + 1];                 // start of each tier's slice of the list
  uint32_t queue_head[kMaxTiers];                    // work-queue heads of the encode kernels
  uint32_t fallback_range[2];                        // {0, items the lane-per-segment kernel passed on}
  uint32_t unfolded_count[kMaxTiers];                // items of each tier that are left to the kernel of the longest ones
  uint32_t unused;
  uint32_t share_head[8][4];                         // items passed on that are claimed; the first word of each
};
static_assert(sizeof(Control) <= 256, "the smallest part of a workspace");

__device__ inline int bin_key(int len, const TierPlan& plan) {
  int lo = 0;
  for (int t = 0; t < plan.n_tiers; ++t) {
    const int cap = plan.cap[t];
    if (len <= cap) {
      // bucket 0 holds the longest strings of the tier
      const int span = cap - lo;
      int b = span > 0 ? (int)(((uint32_t)(cap - len) * (uint32_t)kLenBuckets) / (uint32_t)span) : 0;
      if (b >= kLenBuckets) b = kLenBuckets - 1;
      return t * kLenBuckets + b;
    }
    lo = cap;
  }
  return -1;                                         // longer than any launched variant: skipped
}

// The key of a group of strings or pieces (tier 0).
__device__ inline int group_key(int len) {
  return min((kGroupBytes - min(len, kGroupBytes)) * kLenBuckets / kGroupBytes, kLenBuckets - 1);
}

// What a work item is, stored beside its place in the work list: all that an encode kernel needs to start on it.
struct ItemDesc {
  int64_t begin;                                     // first byte of the item in `bytes`
  int32_t len;                                       // its length in bytes
  int32_t item;                                      // string index, or slot index when strings are split
};

// The work list of a batch whose strings are not split and that has more of them than are resident at once: groups of
// neighbouring strings, longest length bucket first.  (Such a batch has one tier.)  An item costs its wave some ten
// microseconds of round trips whatever its length, so short strings go together: 20,011 strings of up to 400 bytes
// were 105 us one by one and 48 in groups (that kernel; the whole call takes 44 now).  Every 64 strings are divided by one wave, first come first served: a group
// takes strings until the next one would end more than `room` bytes after its beginning.  (With groups of all strings
// that start in one window of the text, which need no walk, items were a third smaller.)
//
// Workgroup b owns the strings [b stretch, (b + 1) stretch), whole tiles of 1,024.  bin_count_kernel leaves each
// stretch's histogram of the length buckets in `part` (kLenBuckets words per workgroup); bin_scatter_kernel adds up
// everybody's, which is at most kBinGrid rows of 256 bytes, so it knows where each bucket begins and where its own part
// of it does, and needs no atomics on memory.  What bounds them is latency, a chain of a few loads each (20,011 strings:
// 4.4 and 5.0 us); one workgroup that walks the batch twice took 1.3 us per 1,024 strings (27 us).
constexpr int kBinGrid = 128;
__global__ __launch_bounds__(1024) void bin_count_kernel(const int64_t* offsets, int batch, int64_t stretch, int room,
                                                         uint32_t* part) {
  __shared__ uint32_t hist[kLenBuckets];
  const int t = threadIdx.x;
  const int64_t first = blockIdx.x * stretch, last = min(first + stretch, (int64_t)batch);
  if (t < kLenBuckets) hist[t] = 0;
  __syncthreads();
  for (int64_t tile = first; tile < last; tile += 1024) {
    const StringGroup g = string_group(offsets, tile, batch, room);
    if (g.members) atomicAdd(&hist[group_key(g.len)], 1u);
  }
  __syncthreads();
  if (t < kLenBuckets) part[blockIdx.x * kLenBuckets + t] = hist[t];
}
// Also resets the work-queue heads.
__global__ __launch_bounds__(1024) void bin_scatter_kernel(const int64_t* offsets, int batch, int64_t stretch,
                                                           int room, Control* c,
                                                           const uint32_t* part, ItemDesc* desc) {
  static_assert(kLenBuckets == 64, "a lane per length bucket");
  __shared__ uint32_t sum_all[16][kLenBuckets], sum_before[16][kLenBuckets];
  __shared__ uint32_t cursor[kLenBuckets];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t all = 0, before = 0;                        // of bucket `lane`: groups, and those of earlier stretches
  for (int b = wave; b < (int)gridDim.x; b += 16) {
    const uint32_t n = part[b * kLenBuckets + lane];
    all += n;
    if (b < (int)blockIdx.x) before += n;
  }
  sum_all[wave][lane] = all;
  sum_before[wave][lane] = before;
  __syncthreads();
  if (wave == 0) {
    for (int w = 1; w < 16; ++w) { all += sum_all[w][lane]; before += sum_before[w][lane]; }
    uint32_t upto = all;                               // inclusive scan over the buckets
    for (int step = 1; step < 64; step <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)upto, step, 64);
      if (lane >= step) upto += o;
    }
    cursor[lane] = upto - all + before;
    const uint32_t total = (uint32_t)__shfl((int)upto, 63, 64);
    if (blockIdx.x == 0) {
      if (lane <= kMaxTiers) c->tier_base[lane] = lane == 0 ? 0u : total;
      if (lane < kMaxTiers) c->queue_head[lane] = 0;
      if (lane < 2) c->fallback_range[lane] = 0;
      if (lane < 8) c->share_head[lane][0] = 0;
    }
  }
  __syncthreads();
  const int64_t first = blockIdx.x * stretch, last = min(first + stretch, (int64_t)batch);
  for (int64_t tile = first; tile < last; tile += 1024) {
    const StringGroup g = string_group(offsets, tile, batch, room);
    if (g.members)
      desc[atomicAdd(&cursor[group_key(g.len)], 1u)] =
          ItemDesc{g.begin, g.len | (g.members << kGroupShift), (int)(tile + t)};
  }
}

// out_offsets[i] = sum of counts[0..i), out_offsets[batch] = total.  A workgroup owns a stretch of strings (whole
// tiles of 1024; the host picks one tile, and more once that would be over kOffsetsGrid workgroups).  It sums the
// counts before its stretch itself, sixteen strings' loads in flight per thread -- they come from L2, 4 bytes per
// string -- so no workgroup waits for another.  What bounds it is those loads' latency: with one workgroup walking
// the whole batch, a tile cost 1.5 us one after the other (20,011 strings: 30 us).
constexpr int kOffsetsGrid = 256;
__global__ __launch_bounds__(1024) void offsets_scan_kernel(const int32_t* counts, int batch, int stretch,
                                                            int64_t* out_offsets) {
  __shared__ int64_t wave_sum[16];
  __shared__ int64_t carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int first = (int)min((int64_t)blockIdx.x * stretch, (int64_t)batch);
  const int last = (int)min((int64_t)first + stretch, (int64_t)batch);
  int64_t before = 0;                                  // tokens of all strings before the stretch
  const int4* const quads = (const int4*)counts;       // (`first` is a multiple of 1024, or nothing is left to do)
  const int n_quads = first / 4;
  for (int q = tid; q < n_quads; q += 4 * 1024) {      // the loads are unconditional (index clamped), the test comes after
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = quads[min(q + u * 1024, n_quads - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (q + u * 1024 < n_quads) before += ((int64_t)v[u].x + v[u].y) + ((int64_t)v[u].z + v[u].w);
  }
  for (int step = 32; step >= 1; step >>= 1) before += __shfl_xor(before, step, 64);
  if (lane == 0) wave_sum[wave] = before;
  if (blockIdx.x == 0 && tid == 0) out_offsets[0] = 0;
  __syncthreads();
  int64_t carry = 0;                                   // (the same in all threads)
  for (int w = 0; w < 16; ++w) carry += wave_sum[w];
  __syncthreads();
  for (int base = first; base < last; base += 1024) {
    const int i = base + tid;
    int64_t v = i < last ? (int64_t)counts[i] : 0;
    for (int step = 1; step < 64; step <<= 1) {
      int64_t o = __shfl_up(v, step, 64);
      if (lane >= step) v += o;
    }
    if (lane == 63) wave_sum[wave] = v;
    __syncthreads();
    int64_t at = carry;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    if (i < last) out_offsets[i + 1] = at + v;
    if (tid == 1023) carry_s = at + v;
    __syncthreads();
    carry = carry_s;
    __syncthreads();
  }
}

// The encode kernels number tokens their own way (byte b = b, row r creates 256 + r); a table built over a
// vocabulary carries the vocabulary's id of each, applied where the ids are written to the output.
__device__ inline int32_t vocabulary_id(const int32_t* id_map, int32_t token) {
  return id_map ? id_map[token] : token;
}

// Small batches: offsets and packing in one launch.  Workgroup s sums the counts before its string itself
// (the batch is at most a few thousand strings), writes out_offsets[s] and copies the string's ids.
__global__ __launch_bounds__(256) void scan_pack_kernel(const int32_t* tmp_ids, const int64_t* offsets,
                                                        const int32_t* counts, int batch, int64_t* out_offsets,
                                                        int32_t* out_ids, const int32_t* id_map) {
  __shared__ int64_t wave_sum[4];
  const int s = blockIdx.x;
  int64_t v = 0;
  for (int i = threadIdx.x; i < s; i += 256) v += counts[i];
  for (int step = 32; step >= 1; step >>= 1) v += __shfl_down(v, step, 64);
  if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = v;
  __syncthreads();
  const int64_t dst = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
  const int k = counts[s];
  if (threadIdx.x == 0) {
    out_offsets[s] = dst;
    if (s == batch - 1) out_offsets[batch] = dst + k;
  }
  const int64_t src = offsets[s];
  for (int i = threadIdx.x; i < k; i += 256) out_ids[dst + i] = vocabulary_id(id_map, tmp_ids[src + i]);
}

// One wave per group of strings: copy its ids from the staging area to the dense output, four rows of 64 loads in
// flight.  A group's ids lie together on both sides; those of a group marked kGroupApart lie string by string in the
// staging area, so lane m keeps what lies between string m's two places and each id looks its string up among them:
// string by string would be a chain of loads each, and such a group may have 64.  What bounds it is the loads' latency:
// 20,011 rows of up to 400 bytes 4.8 us; 100,000 of up to 60 bytes, nearly all groups with a marked string, 6.9 us.
__global__ __launch_bounds__(256) void pack_kernel(const int32_t* tmp_ids, const int64_t* offsets,
                                                   const int64_t* out_offsets, const Control* c, const ItemDesc* desc,
                                                   int32_t* out_ids, const int32_t* id_map) {
  const int lane = threadIdx.x & 63;
  const uint32_t n_groups = c->tier_base[1];
  for (uint32_t g = blockIdx.x * 4 + (threadIdx.x >> 6); g < n_groups; g += gridDim.x * 4) {
    const ItemDesc d = desc[g];
    const int members = (d.len >> kGroupShift) & kGroupMask;
    const bool apart = (d.len & kGroupApart) != 0;     // (per wave: uniform)
    const int64_t src = d.begin, dst = out_offsets[d.item];
    const int k = (int)(out_offsets[d.item + members] - dst);
    int first = 0x7FFFFFFF, lack = 0;                  // string `lane`: its first id in the group, and how far from
    if (apart && lane < members) {                     //   that place in the staging area it lies
      first = (int)(out_offsets[d.item + lane] - dst);
      lack = (int)(offsets[d.item + lane] - src) - first;
    }
    for (int i0 = 0; i0 < k; i0 += 256) {
      int32_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 64 * u + lane;
        int64_t from = src + i;
        if (apart) {
          int m = 0;                                   // the last string whose first id is i or before it
#pragma unroll
          for (int step = 32; step >= 1; step >>= 1)
            if (__shfl(first, m + step, 64) <= i) m += step;
          from += __shfl(lack, m, 64);
        }
        v[u] = i < k ? tmp_ids[from] : 0;              // (token 0 exists in every table)
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 64 * u + lane;
        if (i < k) out_ids[dst + i] = vocabulary_id(id_map, v[u]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Listing the pieces of long strings (piece_slots.h), packing their ids.

// The pieces of a batch's strings and the histogram of their items' keys.  A wave takes 63 slots at a time and looks at one
// more, where its last piece may end; its 64 lanes hold the strings they can belong to.  Pieces that one wave can take
// (tier 0) go together while they lie within `room` bytes, like short strings do, whichever strings they are of; a longer
// one is an item of its own.  The slots that a piece runs over are void; piece_len tells each how many slots back its
// piece starts (negative), so that the packing kernel can give it a share of the copying.  (Other void slots hold 0.)
// item_len: what the list will hold of the item that begins in a slot, an ItemDesc's len for tier 0, minus the length for
// the others, 0 for none.
// Each workgroup leaves its histogram in `part`, from which the next kernel, with the same workgroups, knows where each key
// begins and where its own part of it does: no atomics on memory, and nothing to clear.  What bounds them is latency: some
// ten dependent reads.  8,192 strings of 4 KiB: 11 and 6 us, where numbering the slots, finding the cuts, the histogram, its
// scan and the list were five kernels and 42 us.
constexpr int kListGrid = 256;
__global__ __launch_bounds__(1024) void piece_list_kernel(const uint8_t* bytes, const int64_t* offsets, int batch,
                                                          const uint32_t* cut_bits, const uint8_t* cover, int piece_target,
                                                          int max_string, TierPlan plan, int room, uint32_t n_slots,
                                                          uint32_t steps_each, int32_t* slot_string, int64_t* piece_begin,
                                                          int32_t* piece_len, int32_t* item_len, int32_t* counts,
                                                          int32_t* group_ids, uint32_t* part) {
  __shared__ __align__(16) uint32_t cuts[2048];
  __shared__ uint32_t hist[kBinKeys];
  __shared__ int32_t string_at[16][64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t < 512) ((uint4*)cuts)[t] = ((const uint4*)cut_bits)[t];
  if (t < kBinKeys) hist[t] = 0;
  __syncthreads();
  const uint32_t first_step = (blockIdx.x * 16u + (uint32_t)wave) * steps_each;
  int s0 = 0;                                          // the string of the step's first slot (uniform)
  for (uint32_t step = 0; step < steps_each; ++step) { // uniform
    const uint32_t g0 = (first_step + step) * kListSlots;
    if (g0 >= n_slots) break;                          // uniform
    if (step == 0) s0 = wave_last_string(batch, [&](int i) { return slot_base(offsets[i], i, piece_target) <= g0; });
    const StepSlot slot = step_slots(bytes, offsets, batch, cover, cuts, piece_target, max_string, n_slots, g0, s0,
                                     string_at[wave], slot_string, piece_begin, piece_len);
    const uint32_t g = g0 + (uint32_t)lane;
    const int key = slot.start >= 0 && lane < kListSlots ? bin_key(slot.len, plan) : -1;
    const bool single = key >= 0 && key < kLenBuckets;
    const StringGroup group = group_members(slot.start, slot.start + slot.len, !single, (int)min(n_slots - g0, (uint32_t)kListSlots), room);
    const int item_key = !single ? key : group.members ? group_key(group.len) : -1;
    if (item_key >= 0) atomicAdd(&hist[item_key], 1u);
    if (g < n_slots && lane < kListSlots) {
      group_ids[g] = -1;
      item_len[g] = item_key < 0 ? 0 : single ? group.len | (group.members << kGroupShift) : -slot.len;
      if (key < 0) counts[g] = 0;                      // void slot, or too long for the launched variants
    }
    s0 = slot.next_s0;
  }
  __syncthreads();
  if (t < kBinKeys) part[blockIdx.x * kBinKeys + t] = hist[t];
}

// The work list, tier-major, longest bucket first.  Also resets the work-queue heads.
__global__ __launch_bounds__(1024) void piece_scatter_kernel(TierPlan plan, uint32_t n_slots, uint32_t slots_each, Control* c,
                                                             const uint32_t* part, const int64_t* piece_begin,
                                                             const int32_t* item_len, int32_t* list, ItemDesc* desc) {
  __shared__ uint32_t sum_all[4][kBinKeys], sum_before[4][kBinKeys];
  __shared__ uint32_t scan[kBinKeys], cursor[kBinKeys];
  const int t = threadIdx.x, k = t & (kBinKeys - 1), quarter = t / kBinKeys;
  uint32_t all = 0, before = 0;                        // of key k: items, and those of earlier workgroups
#pragma unroll 8
  for (int b = quarter; b < (int)gridDim.x; b += 4) {
    const uint32_t n = part[b * kBinKeys + k];
    all += n;
    before += b < (int)blockIdx.x ? n : 0u;
  }
  sum_all[quarter][k] = all;
  sum_before[quarter][k] = before;
  __syncthreads();
  uint32_t total = 0;
  if (t < kBinKeys) {
    for (int q = 0; q < 4; ++q) total += sum_all[q][t];
    scan[t] = total;
  }
  __syncthreads();
  for (int step = 1; step < kBinKeys; step <<= 1) {    // inclusive scan, all threads reach the barriers
    uint32_t v = 0;
    if (t < kBinKeys && t >= step) v = scan[t - step];
    __syncthreads();
    if (t < kBinKeys) scan[t] += v;
    __syncthreads();
  }
  if (t < kBinKeys) cursor[t] = scan[t] - total + sum_before[0][t] + sum_before[1][t] + sum_before[2][t] + sum_before[3][t];
  if (blockIdx.x == 0) {
    if (t <= kMaxTiers) c->tier_base[t] = t == 0 ? 0 : scan[(t <= plan.n_tiers ? t : plan.n_tiers) * kLenBuckets - 1];
    if (t < kMaxTiers) c->queue_head[t] = c->unfolded_count[t] = 0;
    if (t < 2) c->fallback_range[t] = 0;
    if (t < 8) c->share_head[t][0] = 0;
  }
  __syncthreads();
  const uint32_t first = blockIdx.x * slots_each, last = min(first + slots_each, n_slots);
  for (uint32_t g = first + (uint32_t)t; g < last; g += 1024u) {
    const int32_t len = item_len[g];
    if (len == 0) continue;
    const uint32_t at = atomicAdd(&cursor[len > 0 ? group_key(len & kGroupLen) : bin_key(-len, plan)], 1u);
    list[at] = (int32_t)g;
    desc[at] = ItemDesc{piece_begin[g], len > 0 ? len : -len, (int32_t)g};
  }
}

// A small batch (small_batch_fits) is not listed: each wave of the encode kernel takes a slot and finds its piece itself
// (slot_piece).  It leaves what is to be done with the piece, for the kernel that comes after.
enum { kSlotDone, kSlotLeft };
// Token offsets of the slots: per-tile sums, then the scan inside each tile.
constexpr int kScanTile = 4096;

__global__ __launch_bounds__(1024) void tile_sum_kernel(const int32_t* counts, uint32_t n_slots, int64_t* tile_sum) {
  __shared__ int64_t wave_sum[16];
  const uint32_t base = blockIdx.x * kScanTile;
  int64_t v = 0;
  for (int j = 0; j < kScanTile / 1024; ++j) {
    const uint32_t g = base + j * 1024 + threadIdx.x;
    if (g < n_slots) v += counts[g];
  }
  for (int step = 32; step >= 1; step >>= 1) v += __shfl_down(v, step, 64);
  if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int w = 0; w < 16; ++w) t += wave_sum[w];
    tile_sum[blockIdx.x] = t;
  }
}

// (Each workgroup adds up the tiles before its own: there is one per 4,096 slots.)
__global__ __launch_bounds__(1024) void slot_offsets_kernel(const int32_t* counts, uint32_t n_slots, const int64_t* tile_sum,
                                                            const int32_t* slot_string, int64_t* slot_out,
                                                            int64_t* out_offsets, int batch) {
  __shared__ int64_t wave_sum[16];
  __shared__ int64_t carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t before = 0;
  for (int i = tid; i < (int)blockIdx.x; i += 1024) before += tile_sum[i];
  for (int step = 32; step >= 1; step >>= 1) before += __shfl_xor(before, step, 64);
  if (lane == 0) wave_sum[wave] = before;
  __syncthreads();
  if (tid == 0) {
    int64_t t = 0;
    for (int w = 0; w < 16; ++w) t += wave_sum[w];
    carry_s = t;
  }
  __syncthreads();
  for (int j = 0; j < kScanTile / 1024; ++j) {
    const uint32_t g = blockIdx.x * kScanTile + j * 1024 + tid;
    const int64_t m = g < n_slots ? (int64_t)counts[g] : 0;
    int64_t v = m;
    for (int step = 1; step < 64; step <<= 1) {
      const int64_t o = __shfl_up(v, step, 64);
      if (lane >= step) v += o;
    }
    if (lane == 63) wave_sum[wave] = v;
    __syncthreads();
    int64_t at = carry_s + v - m;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    if (g < n_slots) {
      slot_out[g] = at;
      const int s = slot_string[g];
      if (s >= 0) out_offsets[s] = at;                 // a string starts at its first slot
    }
    __syncthreads();
    if (tid == 1023) carry_s = at + m;
    __syncthreads();
  }
  if (blockIdx.x == gridDim.x - 1 && tid == 0) out_offsets[batch] = carry_s;
}

// ---------------------------------------------------------------------------------------------------
// Special tokens (section 4.1: special-character lookups before any merging).  The set is small (at most 64
// strings of at most 64 bytes) and, by construction of the set, occurrences cannot overlap, so every byte
// position can decide on its own whether an occurrence starts there: the longest special that matches.

constexpr int kMaxSpecials = 64, kMaxSpecialBytes = 64;

struct SpecialSet {
  uint32_t first_byte[8];                              // bit b: some special starts with byte b
  int32_t n;
  int32_t len[kMaxSpecials];
  uint8_t text[kMaxSpecials][kMaxSpecialBytes];
};

// A workgroup writes the marks of kMarkBlock consecutive bytes, each once and 16 bytes a lane: it collects them in LDS,
// for which it also looks at the kMaxSpecialBytes positions before its stretch, where an occurrence that reaches into
// it can start.  What bounds it is the text and the marks themselves, as long as a byte that starts a special, or looks
// like it, waits for no memory: every byte asks an LDS bit set, a hit is compared with the set's texts four bytes at a
// time, all from LDS, and the string that holds a full match is searched only among the strings of the workgroup's own
// stretch, which two of its waves look up once and whose ends come to LDS.  One chunk a
// thread: with four, a wave works off four times the hits one after the other (2.5 MB of conversations: 30 us instead
// of 13).  54 MB with a special at every 600th byte: about 70 us; with the marks cleared by a kernel before and written
// byte by byte, strings searched in memory: 90 us; one byte a thread with a search over the whole batch: 379 us.
constexpr int kMarkText = 256 * 16;                    // bytes whose occurrences a workgroup looks for
constexpr int kMarkBlock = kMarkText - kMaxSpecialBytes;
constexpr int kMarkWords = (kMarkText + kMaxSpecialBytes) / 4;
constexpr int kMarkStrings = 255;                      // string ends kept in LDS; more (short strings) stay in memory
__global__ __launch_bounds__(256) void special_mark_kernel(const uint8_t* bytes, const int64_t* offsets, int batch,
                                                           int64_t total_bytes, const SpecialSet* set,
                                                           uint8_t* cover) {
  static_assert(kMarkBlock % 16 == 0 && kMaxSpecialBytes % 16 == 0, "chunks of 16 bytes");
  __shared__ __align__(16) uint32_t text[kMarkWords + 4];
  __shared__ __align__(16) uint32_t marks[kMarkBlock / 4];
  __shared__ uint32_t special[kMaxSpecials * kMaxSpecialBytes / 4];
  __shared__ uint32_t first_byte[8];
  __shared__ int32_t length[kMaxSpecials];
  __shared__ int32_t string_begin[kMarkStrings + 1];
  __shared__ int first_string, last_string;
  const int tid = threadIdx.x;
  const int n_specials = set->n;
  const int64_t base = (int64_t)blockIdx.x * kMarkBlock;         // the first byte that this workgroup marks ...
  const int64_t start = base - kMaxSpecialBytes;                 // ... and the first that it looks at
  const int64_t end = min(base + kMarkBlock, total_bytes);
  if (tid < 8) first_byte[tid] = set->first_byte[tid];
  if (tid < n_specials) length[tid] = set->len[tid];
  for (int i = tid; i < n_specials * (kMaxSpecialBytes / 4); i += 256)
    special[i] = ((const uint32_t*)set->text)[i];      // (unused bytes of a text are zero)
  // 16 bytes of the text from position p on, zeros before its beginning and past its end.  Wide loads need the
  // pointer's alignment; without it, and at the end of the text, bytes are read one by one.
  const bool aligned = ((uintptr_t)bytes & 15u) == 0;
  auto chunk_at = [&](int64_t p) {
    if (p < 0) return make_uint4(0, 0, 0, 0);          // (a whole chunk: `start` is a multiple of 16)
    if (aligned && p + 16 <= total_bytes) return *(const uint4*)(bytes + p);
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (p + j < total_bytes) w[j >> 2] |= (uint32_t)bytes[p + j] << (8 * (j & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
  };
  const uint4 mine = chunk_at(start + 16 * tid);
  *(uint4*)&text[4 * tid] = mine;
  if (tid < kMaxSpecialBytes / 16) *(uint4*)&text[kMarkText / 4 + 4 * tid] = chunk_at(start + kMarkText + 16 * tid);
  if (tid == 0) text[kMarkWords] = 0;
  if (tid < kMarkBlock / 16) *(uint4*)&marks[4 * tid] = make_uint4(0, 0, 0, 0);
  if (tid >= 128 && tid < 192) {
    const int s = wave_last_string(batch, [&](int i) { return offsets[i] <= max(start, (int64_t)0); });
    if (tid == 128) first_string = s;
  } else if (tid >= 192) {
    const int s = wave_last_string(batch, [&](int i) { return offsets[i] <= end - 1; });
    if (tid == 192) last_string = s;
  }
  __syncthreads();
  const int s0 = first_string, s1 = last_string;
  const bool ends_here = s1 - s0 < kMarkStrings;       // uniform
  // (positions relative to `start`, clamped far outside the stretch: only comparisons and short rooms are asked)
  if (ends_here && tid <= s1 - s0 + 1)
    string_begin[tid] = (int32_t)min(max(offsets[s0 + tid] - start, (int64_t)-(1 << 28)), (int64_t)1 << 28);
  __syncthreads();
  const uint32_t own[4] = {mine.x, mine.y, mine.z, mine.w};
  const int64_t left = total_bytes - start - 16 * tid; // bytes of the text from my first one on
  uint32_t hits = 0;                                   // bit j: my byte j could start a special
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t b = (own[j >> 2] >> (8 * (j & 3))) & 0xFFu;
    hits |= ((first_byte[b >> 5] >> (b & 31u)) & 1u) << j;
  }
  if (left < 16) hits &= left > 0 ? (1u << (int)left) - 1u : 0u;
  if (start + 16 * tid < 0) hits = 0;
  while (hits) {
    const int at = 16 * tid + __builtin_ctz(hits);     // in the workgroup's text
    hits &= hits - 1u;
    const int64_t p = start + at;
    // byte differences between word w of special i and the text from `at` on, as far as the special goes
    auto differs = [&](int i, int w, int len) {
      const uint32_t here = __builtin_amdgcn_alignbit(text[(at >> 2) + w + 1], text[(at >> 2) + w], 8u * (at & 3));
      const uint32_t word = here ^ special[i * (kMaxSpecialBytes / 4) + w];
      return len - 4 * w >= 4 ? word : word & ((1u << (8 * (len - 4 * w))) - 1u);
    };
    int64_t room = -1;                                 // bytes from p to the end of its string, once they are asked for
    int best = -1, best_len = 0;
    for (int i = 0; i < n_specials; ++i) {
      const int len = length[i];
      if (len <= best_len || p + len > total_bytes) continue;
      int w = 0;
      while (4 * w < len && !differs(i, w, len)) ++w;
      if (4 * w < len) continue;
      if (room < 0) {                                  // the string that holds p: last s with offsets[s] <= p
        if (ends_here) {
          int lo = 0, hi = s1 - s0;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (string_begin[mid] <= at) lo = mid; else hi = mid - 1;
          }
          room = max(string_begin[lo + 1] - at, 0);
        } else {
          int lo = s0, hi = s1;
          while (lo < hi) {
            const int mid = lo + ((hi - lo + 1) >> 1);
            if (offsets[mid] <= p) lo = mid; else hi = mid - 1;
          }
          room = max(offsets[lo + 1] - p, (int64_t)0);
        }
      }
      if (len <= room) { best = i; best_len = len; }
    }
    if (best >= 0) {
      const int to = at - kMaxSpecialBytes;            // in the workgroup's marks
      for (int j = 0; j < best_len; ++j)
        if ((uint32_t)(to + j) < (uint32_t)kMarkBlock)
          ((uint8_t*)marks)[to + j] = (uint8_t)(j == 0 ? kCoverFirst | (uint32_t)best : kCoverRest);
    }
  }
  __syncthreads();
  // (whole chunks: the marks' buffer is padded beyond the text)
  if (tid < kMarkBlock / 16 && base + 16 * tid < total_bytes)
    *(uint4*)(cover + base + 16 * tid) = *(const uint4*)&marks[4 * tid];
}

// Copy every piece's ids to their place in the dense output.  A piece has a few hundred ids, so what limits
// this kernel is how many loads are in flight: a wave takes two slots at a time, reads the next two descriptors
// while it copies, and issues four rows of loads per slot -- and, where the ids are a vocabulary's, their look-ups --
// before the first store.  A slot copies at most kPackShare ids; what a longer piece has beyond them is copied by the
// void slots it runs over, kPackShare each: a piece over m slots has at most (m - 1) * piece target + 1024 bytes.
// 256 pieces of 64 KiB, 41,000 ids each: 121 us with one wave a piece, 18 us so (whole call 443 -> 346 us).
constexpr int kPackShare = 1024;
struct PackItem {
  uint32_t g;
  int k, group;                                        // the piece's own ids, and group_ids
  int64_t src, dst;
};
__device__ inline PackItem pack_item(uint32_t g, uint32_t n_slots, const int64_t* piece_begin, const int32_t* counts,
                                     const int32_t* group_ids, const int64_t* slot_out) {
  PackItem it{g, 0, -1, 0, 0};
  if (g < n_slots) {
    it.k = counts[g];
    it.group = group_ids[g];
    it.src = piece_begin[g];
    it.dst = slot_out[g];
  }
  return it;
}
// A void slot turned into its share of the piece that runs over it, and a piece cut to its own share -- or grown to its
// item, whose ids lie together (2 Ki at most).
__device__ inline void pack_share(PackItem& it, const int64_t* piece_begin, const int32_t* piece_len,
                                  const int32_t* counts, const int64_t* slot_out) {
  if (it.src < 0) {                                    // (per wave: uniform)
    const int back = piece_len[it.g];
    if (back < 0) {
      const uint32_t owner = it.g + (uint32_t)back;
      const int skip = -back * kPackShare;
      it.k = counts[owner] - skip;
      it.src = piece_begin[owner] + skip;
      it.dst = slot_out[owner] + skip;
    }
  }
  it.k = it.group >= 0 ? it.group : min(it.k, kPackShare);
}
__global__ __launch_bounds__(256) void piece_pack_kernel(const int32_t* tmp_ids, uint32_t n_slots,
                                                         const int64_t* piece_begin, const int32_t* piece_len,
                                                         const int32_t* counts, const int32_t* group_ids,
                                                         const int64_t* slot_out, int32_t* out_ids,
                                                         const int32_t* id_map) {
  const int lane = threadIdx.x & 63;
  const uint32_t stride = gridDim.x * 4;               // slots one round of the grid takes: wave w takes w and w + stride
  uint32_t g = blockIdx.x * 4 + (threadIdx.x >> 6);
  PackItem a = pack_item(g, n_slots, piece_begin, counts, group_ids, slot_out);
  PackItem b = pack_item(g + stride, n_slots, piece_begin, counts, group_ids, slot_out);
  while (g < n_slots) {
    const uint32_t g_next = g + 2 * stride;
    const PackItem a_next = pack_item(g_next, n_slots, piece_begin, counts, group_ids, slot_out);
    const PackItem b_next = pack_item(g_next + stride, n_slots, piece_begin, counts, group_ids, slot_out);
    pack_share(a, piece_begin, piece_len, counts, slot_out);
    pack_share(b, piece_begin, piece_len, counts, slot_out);
    const int longest = max(a.k, b.k);                 // (per wave: uniform)
    for (int i0 = 0; i0 < longest; i0 += 256) {
      int32_t va[4], vb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 64 * u + lane;
        va[u] = i < a.k ? tmp_ids[a.src + i] : 0;
        vb[u] = i < b.k ? tmp_ids[b.src + i] : 0;
      }
      if (id_map) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          va[u] = id_map[va[u]];                       // (token 0 exists in every table)
          vb[u] = id_map[vb[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 64 * u + lane;
        if (i < a.k) out_ids[a.dst + i] = va[u];
        if (i < b.k) out_ids[b.dst + i] = vb[u];
      }
    }
    g = g_next;
    a = a_next;
    b = b_next;
  }
}

// Offsets and packing of a batch of at most kSmallSlots slots in one launch: a workgroup sums the counts before its four
// slots itself, four loads of 16 bytes a thread at most, and each of its waves copies one.
__global__ __launch_bounds__(256) void small_pack_kernel(const int32_t* tmp_ids, int n_slots, const int32_t* slot_string,
                                                         const int64_t* piece_begin, const int32_t* piece_len,
                                                         const int32_t* counts, int64_t* out_offsets, int batch,
                                                         int32_t* out_ids, const int32_t* id_map) {
  __shared__ int32_t wave_sum[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int g = 4 * (int)blockIdx.x + wave;
  int32_t before = 0;
  for (int q = t; q < (int)blockIdx.x; q += 256) {
    const int4 v = ((const int4*)counts)[q];
    before += (v.x + v.y) + (v.z + v.w);
  }
  for (int step = 32; step >= 1; step >>= 1) before += __shfl_xor(before, step, 64);
  if (lane == 0) wave_sum[wave] = before;
  int k = 0, own = 0;                                  // this slot's ids, and those of the workgroup's slots before it
  for (int w = 0; w <= wave; ++w) {
    const int n = 4 * (int)blockIdx.x + w < n_slots ? counts[4 * blockIdx.x + w] : 0;
    if (w < wave) own += n; else k = n;
  }
  __syncthreads();
  if (g >= n_slots) return;
  int64_t dst = (int64_t)wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3] + own;
  const int s = slot_string[g];
  if (lane == 0) {
    if (s >= 0) out_offsets[s] = dst;                  // a string starts at its first slot
    if (g == n_slots - 1) out_offsets[batch] = dst + k;
  }
  int64_t src = piece_begin[g];
  if (src < 0) {                                       // a void slot: its share of the piece that runs over it, whose ids end here
    const int back = piece_len[g];
    if (back < 0) {
      const int skip = -back * kPackShare;
      const int all = counts[g + back];
      dst += skip - all;
      src = piece_begin[g + back] + skip;
      k = all - skip;
    }
  }
  k = min(k, kPackShare);
  for (int i0 = 0; i0 < k; i0 += 256) {
    int32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 64 * u + lane;
      v[u] = i < k ? tmp_ids[src + i] : 0;             // (token 0 exists in every table)
    }
    if (id_map) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = id_map[v[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 64 * u + lane;
      if (i < k) out_ids[dst + i] = v[u];
    }
  }
}

}  // namespace bpe
