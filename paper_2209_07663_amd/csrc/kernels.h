// Host-side launchers of the table's kernels (internal to the library).
#pragma once

#include "common.h"
#include "profile.h"

namespace mono {

// Per-call scratch for the update path, carved out of the table's arena.
struct UpdateWorkspace {
  uint32_t* unit_bag;   // [max_ids]: (radix passes) first [sort_units] words: the bag that holds each unit's first occurrence
                        // (a restore call borrows the whole array for its per-record results)
  uint2* pair_a;        // [max_ids] (row, bag) pairs, ping
  uint2* pair_b;        // [max_ids] pong
  uint32_t* hist;       // [sort_hist_words(max_ids)]: digit histograms (per unit, per group), then the bin totals
  float* part;          // [2 * tiles * dim] partial gradient sums of runs that cross tile borders
  uint32_t* part_row;   // [2 * tiles] row (+ head flag) of each partial, kNoRow if unused
  uint64_t tiles;       // what part and part_row are for
};

// How the pairs of a batch are grouped by row.  At most kSortSmall of them are sorted by one block in LDS, in one launch, unless
// they have more than kSortSmallBags bags, which that block would have to walk all by itself; up to kSplitMost, and few pairs
// of many bags, are split and sorted by bucket, in two launches (below); more are sorted by radix passes.  (One block or
// split: steps of 2.3 and 3 K pairs 42.5 and 43.6, 37.5 and 40.3 us, of 4.3 K 52 and 49, of 7.1 K 51 and 45.  Updates of 4 K
// pairs in 40 K and a million bags, 600 K rows in use, by radix passes over units of 512 pairs and split: 41 and 28 us, 134 and
// 125; 17 M rows in use 82 and 28.)
constexpr uint64_t kSortSmall = 4096, kSortSmallBags = 1u << 14;
inline bool sorts_in_one_block(uint64_t n, uint64_t n_bags) { return n <= kSortSmall && n_bags <= kSortSmallBags; }
// The radix passes come in two shapes, chosen per call by the host from its bound on the rows in use:
//   narrow  digits of at most 8 bits, blocks of 256 threads: three passes up to 2^24 rows
//   wide    digits of at most 9 bits, blocks of 512 threads: three passes up to 2^27 rows, where narrow needs four.
//           A wide pass takes a quarter longer than a narrow one (measured on 6.8 M pairs), so wide is taken only
//           where it saves a pass: 1.33 -> 1.30 ms per step on the streaming workload (25 M rows in use), 5.78 ->
//           5.70 ms on the 26 M-ID workload.
// A block owns as many pairs (a unit) as leave it 8 of a bin on average: 2048 and 4096.
struct SortShape {
  uint32_t max_bits, items;
};
constexpr uint32_t kSortNarrowBits = 8, kSortWideBits = 9, kSortNarrowItems = 2048, kSortWideItems = 4096;
constexpr uint32_t kSortNarrowMaxRows = 1u << 24;  // beyond this many rows in use the wide shape saves a pass
constexpr SortShape sort_shape_for(uint32_t hwm_bound) {
  return hwm_bound > kSortNarrowMaxRows ? SortShape{kSortWideBits, kSortWideItems} : SortShape{kSortNarrowBits, kSortNarrowItems};
}
// Pairs of a tile of the reduction: kReduceTile, halved while that leaves fewer than kTilesWanted tiles, as long as a
// lane group (gpb of them in a block) keeps eight pairs to have in flight together.
// (Large tiles only hold more LDS and leave fewer blocks to a compute unit: seg_reduce + combine of 5.8 M pairs of
// dim 32 take 225 / 228 / 214 / 220 us with tiles of 4096 / 2048 / 1024 / 512 pairs.)
constexpr uint32_t kReduceTile = 1024;
// (One number for kernels of which 1024 to 2048 blocks run at a time: of rows of 17 to 256 elements 1792 in bf16, seven waves a
// SIMD, 1536 in fp32, and 1024 past the caches.  2048 tiles are a little more than the first, and their last blocks ran alone: a
// million pairs of bf16 dim 64 in 2048 tiles 74 us, in 4096 58.  But not many more than it takes: 690 K of dim 36 in 2700 20
// us, in 5400 25.  Where tiles are as small as they get there is a step beyond the blocks that run at a time all the same.
// Updates of uniform rows, us: fp32 dim 32 in 1524 tiles, 390 K pairs, 49 and in 1563, 400 K, 53, bf16 dim 64 in 1641, 420 K,
// 66 and in 1797, 460 K, 75.)
constexpr uint64_t kTilesWanted = 2560;
inline uint32_t reduce_tile(uint64_t n, uint32_t gpb) {
  const uint32_t least = 8 * gpb < 256 ? 8 * gpb : 256;
  uint32_t tile = kReduceTile;
  while (tile > least && (n + tile - 1) / tile < kTilesWanted) tile >>= 1;
  return tile;
}

#ifndef MONO_NOALLOC_MAX_IDS
#define MONO_NOALLOC_MAX_IDS (1ull << 18)
#endif

constexpr uint64_t sort_units(uint64_t n, uint32_t items) { return (n + items - 1) / items; }
constexpr uint32_t kSortGroupUnits = 4;  // units come in groups (see sort_hist_kernel)
constexpr uint64_t sort_groups(uint64_t n, uint32_t items) { return sort_units(sort_units(n, items), kSortGroupUnits); }
// The split (sort_split.hip) comes in four sizes: pairs of a unit, occurrences drawn (a row drawn kSplitHits times has a bin of its own), most buckets (of
// about 512 pairs, where that is not too many), threads of a block that splits.  The sample has to find what would not
// fit into a bin (8192 pairs, with the bin's other rows): rows of 1.4 % of 512 K pairs, 0.7 % of a million; such a row is
// missed once in 2800 times, one of half that once in fourteen (a bin of 4096 to 8192 pairs costs little: see
// sort_split.hip).  600 K to a million pairs with units of 1024 instead of 2048 (twice the units
// to collect from) take 20 us longer, with blocks of 256 threads instead of 512 5 to 8; 200 K with samples of 512 25 us
// of `bucket` instead of 12 (too large bins).  Four neighbouring rows in a bucket: 60 to 600 K pairs 0 to 3 % of the
// step faster than with one; a million pairs (rows that were handed out together are hot together) 330 and 294 us.
constexpr uint64_t kSplitMost = 1u << 20;
constexpr uint32_t kSplitSizes = 4, kSplitHits = 4, kSplitTurn = 4096;
constexpr uint64_t kSplitUpTo[kSplitSizes] = {1u << 16, 1u << 17, 1u << 19, kSplitMost};
constexpr uint32_t kSplitItems[kSplitSizes] = {512, 512, 1024, 2048}, kSplitSamples[kSplitSizes] = {512, 1024, 1024, 2048};
constexpr uint32_t kSplitBuckets[kSplitSizes] = {256, 256, 512, 1024};
constexpr int kSplitThreads[kSplitSizes] = {256, 256, 256, 512};
struct SplitShape {
  uint32_t size, buckets_log2, group_log2;
};
inline SplitShape split_shape_for(uint64_t n) {
  uint32_t size = 0, lg = 3;
  while (n > kSplitUpTo[size]) ++size;
  while ((512ull << lg) < n && (1u << lg) < kSplitBuckets[size]) ++lg;
  return {size, lg, size < 3 ? 2u : 0u};
}
// Few pairs in more than 32 times as many bags: the split's blocks walk over the bags for a while only, and search the others.
// (Updates, us, walked and searched: 60 pairs in 33 K bags 44 and 29, in a million 1260 and 32; 4096 in 80 K, twenty times as
// many, 31 and 34, in a million 125 and 36.  The search's code alone costs 0.2 to 0.35 us of 20 to 27.)
inline bool split_searches_bags(uint64_t n, uint64_t n_bags) { return n <= kSplitUpTo[0] && n_bags / 32 > n; }
constexpr uint64_t split_words(uint64_t n) {  // shares of all bins in all units and the list of turns, for batches of at most n elements
  uint64_t most = 0;
  for (uint32_t i = 0; i < kSplitSizes && (i == 0 || n > kSplitUpTo[i - 1]); ++i) {
    const uint64_t m = n < kSplitUpTo[i] ? n : kSplitUpTo[i], hot = kSplitSamples[i] / kSplitHits;
    const uint64_t words = sort_units(m, kSplitItems[i]) * (kSplitBuckets[i] + hot) + 2 + 2 * (hot + m / kSplitTurn);
    most = words > most ? words : most;
  }
  return most;
}
// words of the histogram workspace for batches of at most n elements: the shares of a split, or a histogram per unit (in whole
// groups), one per group and the bin totals
constexpr uint64_t sort_hist_words(uint64_t n) {
  uint64_t most = split_words(n);
  if (n > kSplitMost)
    for (const SortShape s : {sort_shape_for(kSortNarrowMaxRows), sort_shape_for(kSortNarrowMaxRows + 1)}) {
      const uint64_t words = ((kSortGroupUnits + 1) * sort_groups(n, s.items) + 1) << s.max_bits;
      most = words > most ? words : most;
    }
  return most;
}
// most tiles that a batch of at most n pairs can be cut into: tiles of fewer than 256 pairs (32 at least) only
// where 256 would make fewer than kTilesWanted of them
inline uint64_t reduce_tiles(uint64_t n) {
  const uint64_t fine = (n + 31) / 32 < 2 * kTilesWanted ? (n + 31) / 32 : 2 * kTilesWanted, coarse = (n + 255) / 256;
  return fine > coarse ? fine : coarse;
}

// How many bits of the row index are sorted, in how many passes (computed alike on host and device).
struct SortPlan {
  uint32_t hwm, bits, passes, per;
  __host__ __device__ uint32_t shift(uint32_t p) const { return p * per; }
  __host__ __device__ uint32_t width(uint32_t p) const { return bits - p * per < per ? bits - p * per : per; }
};
__host__ __device__ inline SortPlan make_sort_plan(uint32_t hwm, uint32_t max_bits) {
  SortPlan s;
  s.hwm = hwm;
  s.bits = 1;
  const uint32_t top = hwm > 0 ? hwm - 1 : 0;  // sorted keys are row indices below hwm (hwm itself marks "dropped")
  while (s.bits < 32 && (top >> s.bits) != 0) ++s.bits;
  s.passes = (s.bits + max_bits - 1) / max_bits;
  s.per = (s.bits + s.passes - 1) / s.passes;
  return s;
}

// What a restore call supplies per record instead of the initial state of a fresh key
// (values == nullptr: an ordinary lookup_or_insert).
struct RestoreSource {
  const float* values;   // [n * dim] fp32, rounded to the storage type on the way in
  const float* acc;      // [n] accumulators
  const uint32_t* seen;  // [n] last-seen steps
};

hipError_t launch_lookup_or_insert(const TableView& t, const int64_t* d_keys, uint64_t n, uint32_t step, uint32_t epoch,
                                   int32_t* d_rows_out, const RestoreSource& src, hipStream_t stream, Profiler* prof);

// Tables without expiry: is a key's counter looked at before its buckets?  A counter below the threshold proves the key
// absent and saves it both bucket lines, but the look costs every stored key a random access.  So it is taken after a call
// in which enough occurrences missed, as about kSampledBlocks blocks of the election saw them:
//   batches of at most kElectSmall  those of keys that their counters kept out, from a 16th of the batch on.  lookup_or_insert
//             of 100 K uniform keys, threshold 3: 18.1 us without the look and 18.9 with it when all are known, 32.1 and
//             30.7 at a tenth absent, 41.4 and 36.3 when all are; 200 K 20.7 / 23.9, 38.7 / 36.3, 53.6 / 48.3.  Keys that
//             are new and admitted at once (threshold 0 or 1) do not count: their insertion reads the buckets anyway, and
//             finds them in the L2 where the probe has just been (200 K new keys 91.7 us without the look, 96.3 with it)
//   larger ones  all that missed, from an eighth on.  What counts is how many distinct keys miss for each distinct one that
//             is found (they break even at about one), and hot IDs are found many times: streams of Zipf IDs, where an
//             eighth to a fifth of the occurrences miss, take 660 us of probes with the look and 730 without (26 M IDs a
//             step, threshold 1) and 200 and 207 (6.8 M, threshold 3).  Evenly spread IDs want the line at a quarter: 4 M
//             keys, threshold 3, 112 us without and 184 with it when all are known, 178 / 215 at a tenth absent, 196 / 218
//             at a fifth, 243 / 234 at 0.3, 384 / 325 at 0.6, 541 / 450 at 1; threshold 1 743 / 684 and 1155 / 1053
constexpr uint64_t kElectSmall = 1u << 19;  // largest batch whose election takes one occurrence per thread, others four
constexpr uint64_t kSampledBlocks = 16;     // (their atomics meet at one word, and hold up the end of a small election)
struct MissSample {
  uint32_t every;   // each `every`th block of the election is looked at; 0: none
  uint64_t enough;  // missing occurrences in those blocks from which on the next call looks at counters first
};
inline MissSample miss_sample(uint64_t n, uint64_t blocks, uint64_t per_block) {
  const uint64_t every = (blocks + kSampledBlocks - 1) / kSampledBlocks, looked_at = (blocks + every - 1) / every;
  const uint64_t sampled = looked_at * per_block < n ? looked_at * per_block : n;
  return {(uint32_t)every, sampled * (n <= kElectSmall ? 1 : 2) / 16 + 1};
}

// The same in one kernel, for batches of at most kSmallLookup keys that are not a restore call.
constexpr uint64_t kSmallLookup = 4096;
hipError_t launch_lookup_small(const TableView& t, const int64_t* d_keys, uint64_t n, uint32_t step, uint32_t epoch,
                               int32_t* d_rows_out, hipStream_t stream, Profiler* prof);

// Re-inserts every element of src into dst (dst empty, same dim and storage type, capacity >= src's),
// carries the free-row stack over and spreads the occurrence counters; rows are copied by the caller.
hipError_t launch_migrate(const TableView& dst, const TableView& src, int32_t src_free_n, hipStream_t stream);

hipError_t launch_gather_pool(const TableView& t, const int32_t* d_rows, uint64_t n, const int64_t* d_offsets,
                              uint64_t n_bags, float* d_out, hipStream_t stream, Profiler* prof);

// Pooled embeddings of the quotient-remainder decomposition: two dense tables of 2^log2_rows rows each.
hipError_t launch_qr_gather_pool(const void* d_rem, const void* d_quot, uint32_t log2_rows, uint32_t dim, bool bf16,
                                 const int64_t* d_ids, uint64_t n, const int64_t* d_offsets, uint64_t n_bags,
                                 float* d_out, hipStream_t stream);

// hwm_bound: a number the table's high-water mark of rows cannot exceed when the call runs (the capacity, or
// less if the host knows better): it decides how many sort passes are launched.
hipError_t launch_apply_grad_adagrad(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                                     const int64_t* d_offsets, uint64_t n_bags, const float* d_grad, float lr, float eps,
                                     uint32_t hwm_bound, hipStream_t stream, Profiler* prof);

// Group the (row, bag) pairs of a batch by row; the result is in pair_b, the number of pairs in the control block's scratch.
// Of a batch that sorts_in_one_block, and of at most kSplitMost pairs.
hipError_t launch_sort_small(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                             const int64_t* d_offsets, uint64_t n_bags, hipStream_t stream, Profiler* prof);
hipError_t launch_split_pairs(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                              const int64_t* d_offsets, uint64_t n_bags, hipStream_t stream, Profiler* prof);

// Stable LSD radix sort of the (row, bag) pairs of a larger batch; the result is in pair_b if the plan for
// the device's high-water mark (digits of at most *max_bits bits) has an odd number of passes, else in pair_a.
// Returns how many passes were queued (those the plan for hwm_bound needs) and the widest digit of the shape used.
hipError_t launch_sort_pairs(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                             const int64_t* d_offsets, uint64_t n_bags, uint32_t hwm_bound, uint32_t* launched,
                             uint32_t* max_bits, hipStream_t stream, Profiler* prof);

// look_all: the noted bounds cannot be relied on, every bucket that holds something is looked at
hipError_t launch_expire_sweep(const TableView& t, uint32_t now, bool look_all, uint64_t* d_n_expired,
                               int64_t* d_expired_keys, uint64_t max_expired, hipStream_t stream, Profiler* prof);

hipError_t launch_export(const TableView& t, int64_t* d_keys, int32_t* d_row, uint32_t* d_last_seen, int64_t* d_slot,
                         uint64_t max_n, bool touched_only, hipStream_t stream);
hipError_t launch_export_values(const TableView& t, const int32_t* d_row, uint64_t n, float* d_values, float* d_acc,
                                hipStream_t stream);

// Scratch of a sorted export of at most n elements: the elements as the scan finds them, and the sort's buffers.
struct ExportWorkspace {
  uint64_t* key[2];          // [n] ping, pong; the scan writes key[0]
  uint32_t* idx[2];          // [n] position of the element in row / seen / slot
  int32_t* row;              // [n]
  uint32_t* seen;            // [n]
  int64_t* slot;             // [n]
  uint32_t* hist;            // [256 * (export_sort_units(n) + 1)]
};
uint64_t export_sort_units(uint64_t n);
// leaves OR and AND of the keys found in the control block's scratch
hipError_t launch_export_bits(const TableView& t, const ExportWorkspace& ws, uint64_t max_n, hipStream_t stream);
// varying: the bits in which the keys differ (of more than kRangesMost of them)
constexpr uint64_t kRangesMost = 1u << 17;
hipError_t launch_export_sort(const ExportWorkspace& ws, uint64_t n, uint64_t varying, int64_t* d_keys, int32_t* d_row,
                              uint32_t* d_last_seen, int64_t* d_slot, hipStream_t stream);

// Cuts every count back to what it is read as (255 at most).  Tables without expiry need it before their counters have
// taken kCountMost occurrences since the last time: a call adds at most 2^28 to each of a key's counters, which may be
// one, so that no count can pass 2^31 + 2^30.  (A look at the counter of every missing key, by the election, guarded the
// counts before: 26 M IDs a step of which 4 M are new 401 us of election with it, 311 without, 6.8 M 141 and 111, 200 K 17.6 and 9.9.)
constexpr uint64_t kCountMost = 1ull << 31;
hipError_t launch_filter_cut(const TableView& t, hipStream_t stream);
hipError_t launch_filter_export(const TableView& t, uint32_t* d_words, uint64_t first, uint64_t count,
                                hipStream_t stream);
// Arrays on their way to the host (see mono_copy_to_host).
constexpr uint32_t kCopyParts = 8;
struct CopyParts {
  const void* from[kCopyParts];
  void* to[kCopyParts];
  uint64_t words[kCopyParts];  // of four bytes
};
hipError_t launch_copy_to_host(const CopyParts& parts, uint32_t n, hipStream_t stream);
hipError_t launch_filter_import(const TableView& t, const uint32_t* d_words, uint64_t first, uint64_t count,
                                hipStream_t stream);
hipError_t launch_table_init(const TableView& t, uint64_t dset_size, hipStream_t stream);

}  // namespace mono
