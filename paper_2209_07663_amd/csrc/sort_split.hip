// Grouping of the (row, bag) pairs of a middle-sized batch in two launches: the occurrences of a row come next to each
// other, in the order of the batch, which is all that the gradient reduction asks for.
//
//   split   a block owns kItems consecutive occurrences, finds their bags and brings them into the order of their bins in
//           LDS; it writes them out as they lie there, and where its share of every bin begins
//   bucket  a block per bin collects the bin's shares of all units (in the order of the units), sorts them by row in LDS
//           and writes them behind those of the bins before it
// Nothing is counted or scanned across the batch in launches of its own: where a bin begins in the result is the sum of
// where it begins in every unit.  (The radix passes that larger batches take are three launches a digit; up to a million
// pairs those are bound by the latency of each.  Both ways, us: 26 K pairs 25-29 and 15, 81 K 33 and 18, 204 K 33 and 25,
// 690 K 48 and 33; whole training steps 83 -> 70, 87 -> 70, 76 -> 63, 172 -> 159, of a million bf16 pairs 316 -> 287.)
//
// Bins must fit into LDS whatever rows the batch holds.  A bin is the upper bits of a bijective hash of the row (four
// neighbouring rows, whose states share a line, stay together), so that rows spread evenly; rows that make up a good part
// of the batch are told from a sample of it and have a bin each, which needs no sort and may be of any size.  Every block
// takes the same sample and comes to the same answer.  A bin that is too large all the same, for a row that the sample has
// missed, is sorted by words of half the size (kBucketWords).  What is larger than that takes rows that someone chose for
// it; such a bin is taken in pieces, by ranges of rows, by its one block: the more pairs, the more ranges and the longer
// each, 0.9 ms for 30 K pairs of one bin, 12 for 120 K, 117 for 500 K, 680 for a million.
//
// Both kernels are chains of dependent steps, ten thousand cycles in all: blocks of few waves (one to a SIMD: instructions
// of several would queue for it; two where a block has 2048 pairs), loads as early as their addresses are known, little
// code (a kernel that runs once waits for its instructions too).  One block that sorts a bin by itself from the row
// indices of the whole batch, in one launch, took 33 us for 26 K pairs.
#include "common.h"
#include "kernels.h"
#include "sort_ops.h"

namespace mono {

// What a row becomes before it is split: its low bits as they are, the upper ones times an odd number (a bijection of
// the `bits` bits of a row index).  The top bits are the bucket, the others order the rows of a bucket.
struct SplitKey {
  uint32_t hwm, low, odd, mask, rest, buckets;
  __device__ SplitKey(uint32_t hwm_, uint32_t buckets_log2, uint32_t group_log2) : hwm(hwm_) {
    const uint32_t bits = hwm > 2 ? 32 - __clz(hwm - 1) : 1, top = bits < buckets_log2 ? bits : buckets_log2;
    rest = bits - top;
    low = rest < 3 ? 0u : (rest - 3 < group_log2 ? rest - 3 : group_log2);  // (eight groups of rows to a bucket, at least)
    const uint32_t high = bits - low;
    odd = (0x9E3779B1u >> (32 - high)) | 1u;
    mask = (1u << high) - 1u;  // (rows are at most 2^30)
    buckets = 1u << top;
  }
  __device__ uint32_t key(uint32_t row) const { return (((row >> low) * odd) & mask) << low | (row & ((1u << low) - 1)); }
  __device__ uint32_t bucket(uint32_t key) const { return key >> rest; }
  __device__ uint32_t inverse() const {  // of `odd`, modulo 2^32: each step doubles the bits that are right
    uint32_t x = odd;
#pragma unroll
    for (int i = 0; i < 4; ++i) x *= 2u - odd * x;
    return x;
  }
  __device__ uint32_t row(uint32_t key, uint32_t inv) const {
    return (((key >> low) * inv) & mask) << low | (key & ((1u << low) - 1));
  }
};

constexpr uint32_t kNoSplitRow = 0xFFFFFFFFu;

// Sample i: one occurrence of every stratum, at a place in it that follows no stride.
template <uint32_t kSamples>
__device__ inline uint32_t sample_at(uint32_t n, uint32_t i) {
  static_assert(kSplitMost * kSamples < 1ull << 32, "a stratum's bounds fit a word");
  const uint32_t first = n * i / kSamples, last = n * (i + 1) / kSamples;  // (never empty)
  return first + __umulhi(i * 0x9E3779B1u, last - first);
}

// Turns in which the pairs of a row that was drawn `hits` times are copied: about kSplitTurn pairs each.  (All rows
// together: no more than hot rows and n / kSplitTurn.)
template <uint32_t kSamples>
__device__ inline uint32_t split_turns(uint32_t hits, uint32_t n) {
  return 1 + (uint32_t)((uint64_t)hits * n / kSamples / kSplitTurn);
}

template <int kBlock, uint32_t kItems, uint32_t kSamples, uint32_t kBuckets, bool kSearch>
__global__ __launch_bounds__(kBlock) void sort_split_kernel(Control* __restrict__ ctl, const int32_t* __restrict__ rows,
                                                            uint32_t n, const int64_t* __restrict__ offsets,
                                                            uint64_t n_bags, uint32_t buckets_log2, uint32_t group_log2,
                                                            uint32_t* __restrict__ shares, uint32_t* __restrict__ turns_n,
                                                            uint2* __restrict__ turns, uint2* __restrict__ dst) {
  constexpr int kWaves = kBlock / 64;
  constexpr uint32_t kPerWave = kItems / kWaves, kRounds = kPerWave / 64, kDrawn = kSamples / kBlock;
  constexpr uint32_t kHot = kSamples / kSplitHits, kBins = kBuckets + kHot;  // no more hot rows, no more bins
  constexpr uint32_t kSeen = 2 * kSamples, kHotSlots = kSamples, kDigit = kBins < 512 ? 9 : (kBins < 1024 ? 10 : 11);
  static_assert(kBins < (1u << kDigit) && kItems <= 0x8000, "ranks and shares fit their words");
  static_assert((kSamples & (kSamples - 1)) == 0 && 2 * kHot <= kHotSlots, "sets are powers of two, and at most half full");
  static_assert(kSamples % kBlock == 0 && kItems % kBlock == 0, "whole rounds of the block");
  union Lds {
    struct {
      uint32_t row[kSeen], hits[kSeen];  // set of the sampled rows, and how often each was drawn
    } seen;
    uint32_t bag_here[kItems];  // then, until the pairs are staged
    uint2 stage[kItems];
  };
  __shared__ Lds s;
  __shared__ __align__(4) uint16_t cnt[kWaves][kBins];
  __shared__ uint32_t hot_row[kHot], hot_hits[kHot], hot_turns[kHot], hot_key[kHotSlots], hot_bin[kHotSlots];
  __shared__ uint32_t n_hot, wave_sum[kWaves], wave_last[kWaves], bags_before[2], bags_left;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
  const uint32_t unit = blockIdx.x, ubase = unit * kItems, uend = ubase + kItems < n ? ubase + kItems : n;
  const uint32_t base = ubase + wave * kPerWave;

  // The bag that holds the unit's first occurrence, or one not far before it: the last one whose offset is not behind.  A
  // thread looks at one bag a step; the steps lie between the barriers of what else is to be done.  (Whatever the offsets
  // hold, `lo` stays below n_bags.)
  uint64_t lo = 0, hi = n_bags;
  const auto not_behind = [&]() {
    const uint64_t step = (hi - lo + kBlock - 1) / kBlock, p = lo + (uint64_t)(tid + 1) * step;
    return p < hi && bounded_offset(offsets, p, n) <= ubase;
  };
  const auto report = [&](bool yes, uint32_t turn) {
    const uint64_t m = __ballot(yes);
    if (lane == 0 && m) atomicAdd(&bags_before[turn], (uint32_t)__popcll(m));
  };
  const auto narrow = [&](uint32_t turn) {
    const uint64_t step = (hi - lo + kBlock - 1) / kBlock, k = bags_before[turn];
    hi = lo + (k + 1) * step < hi ? lo + (k + 1) * step : hi;
    lo += k * step;
  };
  // (The walk over the unit's bags may begin as many bags too early as the block has threads: those say that they begin at the
  // unit's first occurrence, where the last of all that say so counts.)
  const auto near = [&]() { return hi - lo <= (uint64_t)kBlock; };
  // asked for at once: the unit's rows, the sample, the first step of the search
  uint32_t mine[kRounds], drawn[kDrawn];
#pragma unroll
  for (uint32_t q = 0; q < kDrawn; ++q) drawn[q] = (uint32_t)rows[sample_at<kSamples>(n, q * kBlock + tid)];
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) mine[r] = base + r * 64 + lane < n ? (uint32_t)rows[base + r * 64 + lane] : kNoSplitRow;
  bool yes = not_behind();
  const SplitKey split(ctl->hwm, buckets_log2, group_log2);
#pragma unroll
  for (uint32_t b = 0; b < kSeen; b += kBlock) {
    s.seen.row[b + tid] = kNoSplitRow;
    s.seen.hits[b + tid] = 0;
  }
#pragma unroll
  for (uint32_t b = 0; b < kHotSlots; b += kBlock) hot_key[b + tid] = kNoSplitRow;
  static_assert(kWaves * kBins % 2 == 0, "whole words");
  for (uint32_t b = tid; b < kWaves * kBins / 2; b += kBlock) reinterpret_cast<uint32_t*>(cnt)[b] = 0;
  if (tid == 0) n_hot = 0;
  if (kSearch && tid == 0) bags_left = 0;
  if (tid < 2) bags_before[tid] = 0;
  __syncthreads();
  report(yes, 0);
  {
    uint32_t at[kDrawn], old[kDrawn];
#pragma unroll
    for (uint32_t q = 0; q < kDrawn; ++q) {
      at[q] = (drawn[q] * 0x85EBCA6Bu) >> (32 - __builtin_ctz(kSeen));
      old[q] = drawn[q] < split.hwm ? atomicCAS(&s.seen.row[at[q]], kNoSplitRow, drawn[q]) : drawn[q];
    }
#pragma unroll
    for (uint32_t q = 0; q < kDrawn; ++q) {
      while (old[q] != kNoSplitRow && old[q] != drawn[q]) {  // at most half of the slots are ever taken: a free one turns up
        at[q] = (at[q] + 1) & (kSeen - 1);
        old[q] = atomicCAS(&s.seen.row[at[q]], kNoSplitRow, drawn[q]);
      }
      if (drawn[q] < split.hwm) atomicAdd(&s.seen.hits[at[q]], 1u);
    }
  }
  __syncthreads();
  narrow(0);
  const bool found = near();  // (block-uniform)
  if (!found) yes = not_behind();
#pragma unroll
  for (uint32_t b = 0; b < kSeen; b += kBlock)
    if (s.seen.hits[b + tid] >= kSplitHits) {
      const uint32_t i = atomicAdd(&n_hot, 1u);  // (no more than samples / hits)
      hot_row[i] = s.seen.row[b + tid];
      hot_hits[i] = s.seen.hits[b + tid];
    }
  if (!found) report(yes, 1);
  __syncthreads();
  if (!found) narrow(1);
  const uint32_t hot = n_hot, bins = split.buckets + hot;
  if (hot) {  // block-uniform.  Numbered in the order of the rows: the list's own order is that of the block's atomics
    for (uint32_t i = tid; i < hot; i += kBlock) {
      const uint32_t row = hot_row[i];
      uint32_t number = 0;
      for (uint32_t j = 0; j < hot; ++j) number += hot_row[j] < row;
      hot_turns[number] = split_turns<kSamples>(hot_hits[i], n);
      uint32_t at = (row * 0x85EBCA6Bu) >> (32 - __builtin_ctz(kHotSlots));
      while (atomicCAS(&hot_key[at], kNoSplitRow, row) != kNoSplitRow) at = (at + 1) & (kHotSlots - 1);
      hot_bin[at] = split.buckets + number;
    }
    __syncthreads();
  }
  while (!near()) {  // (more bags than the cube of the block's threads)
    if (tid == 0) bags_before[0] = 0;
    __syncthreads();
    report(not_behind(), 0);
    __syncthreads();
    narrow(0);
    __syncthreads();
  }
  // the unit's bags from the one that holds its first occurrence on, neighbouring threads neighbouring bags
  constexpr uint32_t kBagsAhead = 2;
  uint64_t bag = lo + tid;
  uint32_t start[kBagsAhead];
  const auto ask = [&]() {
#pragma unroll
    for (uint32_t q = 0; q < kBagsAhead; ++q) {
      const uint64_t b = bag + q * kBlock;
      start[q] = (uint32_t)(b < n_bags ? bounded_offset(offsets, b, n) : uend);
    }
  };
  ask();
  // rank of every pair among the wave's pairs of its bin, 64 at a time; what is left in `cnt` is the wave's counts
  uint2 kv[kRounds];
  uint32_t rank[kRounds];  // bin << 16 | rank
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    kv[r] = make_uint2(kNoSplitRow, 0u);
    rank[r] = 0;
    if (mine[r] < split.hwm) {
      kv[r].x = split.key(mine[r]);
      rank[r] = split.bucket(kv[r].x);
    }
  }
  if (hot) {
#pragma unroll
    for (uint32_t r = 0; r < kRounds; ++r) {
      uint32_t at = (mine[r] * 0x85EBCA6Bu) >> (32 - __builtin_ctz(kHotSlots)), there = hot_key[at];
      while (there != kNoSplitRow && there != mine[r]) {
        at = (at + 1) & (kHotSlots - 1);
        there = hot_key[at];
      }
      if (there != kNoSplitRow) rank[r] = hot_bin[at];
    }
  }
  {
    uint16_t* off = cnt[wave];
#pragma unroll
    for (uint32_t r = 0; r < kRounds; ++r) {
      const bool valid = kv[r].x != kNoSplitRow;
      const uint32_t bin = rank[r];
      const uint64_t peers = same_digit_lanes<kDigit>(bin, valid);
      const uint32_t before = lanes_before(peers);
      rank[r] = (bin << 16) | (wave_load(off + bin) + before);
      wave_order();
      if (valid && before == 0) wave_store(off + bin, (uint16_t)(rank[r] + (uint32_t)__popcll(peers)));
      wave_order();
    }
  }
  __syncthreads();  // every wave has counted, and nobody needs the sample any more
#pragma unroll
  for (uint32_t p = 0; p < kItems; p += kBlock) s.bag_here[p + tid] = 0;
  constexpr uint32_t kPer = (kBins + kBlock - 1) / kBlock;  // consecutive bins of a thread
  uint32_t c[kPer][kWaves], sum = 0;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      c[q][w] = tid * kPer + q < kBins ? cnt[w][tid * kPer + q] : 0u;
      sum += c[q][w];
    }
  }
  const uint32_t x = wave_sums(sum);
  if (lane == 63) wave_sum[wave] = x;
  __syncthreads();
  uint32_t total = 0, run = x - sum;
#pragma unroll
  for (uint32_t w = 0; w < (uint32_t)kWaves; ++w) {
    if (w < wave) run += wave_sum[w];
    total += wave_sum[w];
  }
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t b = tid * kPer + q, from = run;
    if (b < bins) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        cnt[w][b] = (uint16_t)run;
        run += c[q][w];
      }
      shares[unit * kBins + b] = from | (run - from) << 16;
    }
  }
  if (unit == 0) {  // the turns in which the next kernel copies the hot rows' bins
    for (uint32_t i = tid; i < hot; i += kBlock) {
      uint32_t first = 0;
      for (uint32_t j = 0; j < i; ++j) first += hot_turns[j];
      for (uint32_t j = 0; j < hot_turns[i]; ++j) turns[first + j] = make_uint2(split.buckets + i, j << 16 | hot_turns[i]);
      if (i == hot - 1) turns_n[0] = first + hot_turns[i];
    }
    if (tid == 0) {
      ctl->scratch[kHotBins] = hot;
      if (hot == 0) turns_n[0] = 0;
    }
  }
  // The bag of every occurrence: every bag leaves its number at its first occurrence, an occurrence takes the number left
  // at or before it (as in the radix sort's first pass; whatever the offsets hold, every write stays inside the unit and
  // every bag number that is used is one of the batch).  With kSearch a unit whose occurrences lie in very many bags ends this
  // after kBagTurns turns, of 0.6 us each, and every occurrence searches the other bags, which takes about as long as those turns.
  constexpr uint32_t kBagTurns = 16;
  bool more = true;
  for (uint32_t turn = 0; more && (!kSearch || turn < kBagTurns); ++turn) {
#pragma unroll
    for (uint32_t q = 0; q < kBagsAhead; ++q) {
      const uint64_t b = bag + q * kBlock;
      const uint32_t at = start[q] > ubase ? start[q] - ubase : 0;
      more = b < n_bags && start[q] < uend;
      if (more) atomicMax(&s.bag_here[at], (uint32_t)b + 1u);
    }
    bag += (uint64_t)kBlock * kBagsAhead;
    if (more) ask();
  }
  if (kSearch && more) bags_left = 1;  // (the threads that say so agree)
  __syncthreads();
  uint32_t carry = 0;  // the last number left in the wave's earlier elements
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    const uint32_t mark = s.bag_here[wave * kPerWave + r * 64 + lane];
    kv[r].y = max(wave_maxima(mark), carry);
    carry = lane_value(kv[r].y, 63);
  }
  if (lane == 0) wave_last[wave] = carry;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < wave; ++w) before = wave_last[w] ? wave_last[w] : before;
  const uint32_t last_bag = (uint32_t)(n_bags - 1);
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    const uint32_t b = kv[r].y ? kv[r].y : before;
    kv[r].y = min(b ? b - 1u : 0u, last_bag);
  }
  if constexpr (kSearch) {
    const uint64_t walked = lo + (uint64_t)kBagTurns * kBagsAhead * kBlock;
    if (bags_left && walked < n_bags) {  // block-uniform: how many of the other bags are not behind an occurrence
      const uint32_t left = (uint32_t)(n_bags - walked);
      uint32_t k[kRounds] = {};
      for (uint32_t step = 1u << (31 - __clz(left)); step; step >>= 1) {
#pragma unroll
        for (uint32_t r = 0; r < kRounds; ++r) {
          const uint32_t p = k[r] + step;  // (no more than twice `left`, and a batch has at most 2^28 + 1 bags)
          if (p <= left && bounded_offset(offsets, walked + p - 1, n) <= base + r * 64 + lane) k[r] = p;
        }
      }
#pragma unroll
      for (uint32_t r = 0; r < kRounds; ++r)
        if (k[r]) kv[r].y = (uint32_t)walked + k[r] - 1;
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r)
    if (kv[r].x != kNoSplitRow) s.stage[cnt[wave][rank[r] >> 16] + (rank[r] & 0xFFFFu)] = kv[r];
  __syncthreads();
  for (uint32_t p = tid; p < total; p += kBlock) dst[ubase + p] = s.stage[p];
}

// ---- buckets ---------------------------------------------------------------------------------------

constexpr uint32_t kBucketMost = 4096;  // pairs that a block sorts in LDS
// Twice as many, where a key within the bucket and a place in it fit a word together: the words are sorted then, which take
// half the room, and the bags fetched in their order.  (Of 200 batches each of 524 K and of a million pairs, Zipf 0.9 to 1.5,
// one in six has such a bin, and none a bin of more than 5.6 K; taken in pieces, such a bin held up the update of 400 K
// pairs, dim 128 in bf16, 130 us instead of 102, and of a million, dim 32, 151 instead of 104.)
constexpr uint32_t kPlaceBits = 13, kBucketWords = 1u << kPlaceBits;
constexpr uint32_t kBucketDigit = 8, kBucketBins = 1u << kBucketDigit;
constexpr uint32_t kTogether = 4;  // pairs that a thread asks for at a time

template <int kBlock>
struct BucketLds {
  static constexpr int kWaves = kBlock / 64;
  uint32_t first[kBlock];  // pairs of the bin in the units before this one
  uint16_t from[kBlock];   // where the unit's share of the bin lies in the unit
  union {
    uint16_t cnt[kWaves][kBucketBins];
    uint32_t in_range[kBucketBins];
  };
  union {
    uint2 pairs[kBucketMost];
    uint32_t words[kBucketWords];  // key within the bucket << kPlaceBits | place in the bin
  };
  uint32_t wave_sum[2 * kWaves];
  uint32_t range[3];
};
static_assert(sizeof(BucketLds<512>) <= 160 * 1024 / 4 && kSplitItems[kSplitSizes - 1] < 0x10000, "four blocks to a compute unit");

// The pairs at kTogether places of the bin, which is in the order of the batch; those at places from `end` on are left as they are.
template <int kBlock>
__device__ inline void pairs_at(const BucketLds<kBlock>& s, uint32_t units_pow2, uint32_t items, const uint2* __restrict__ src,
                                const uint32_t (&at)[kTogether], uint32_t end, uint2 (&p)[kTogether]) {
  uint32_t u[kTogether];
#pragma unroll
  for (uint32_t j = 0; j < kTogether; ++j) u[j] = 0;
  for (uint32_t d = units_pow2 >> 1; d > 0; d >>= 1) {
#pragma unroll
    for (uint32_t j = 0; j < kTogether; ++j) u[j] += s.first[u[j] + d] <= at[j] ? d : 0u;
  }
#pragma unroll
  for (uint32_t j = 0; j < kTogether; ++j)
    if (at[j] < end) p[j] = src[u[j] * items + s.from[u[j]] + (at[j] - s.first[u[j]])];
}
// q, q + step, ...
template <int kBlock>
__device__ inline void pairs_of_bin(const BucketLds<kBlock>& s, uint32_t units_pow2, uint32_t items,
                                    const uint2* __restrict__ src, uint32_t q, uint32_t step, uint32_t end,
                                    uint2 (&p)[kTogether]) {
  uint32_t at[kTogether];
#pragma unroll
  for (uint32_t j = 0; j < kTogether; ++j) at[j] = q + j * step;
  pairs_at(s, units_pow2, items, src, at, end, p);
}

__device__ inline uint32_t sort_key(uint2 pair) { return pair.x; }
__device__ inline uint32_t sort_key(uint32_t word) { return word >> kPlaceBits; }

// Stable sort of `count` elements by the low `bits` bits of their keys, into `room`.  A wave owns 64 * rounds consecutive ones;
// they are in registers: e[r] of lane l is the wave's element 64 r + l.  A digit is one walk over them, which ranks; what it leaves behind
// are the waves' counts.
template <int kBlock, typename T, uint32_t kRounds>
__device__ inline void sort_bucket(BucketLds<kBlock>& s, T (&e)[kRounds], T* room, uint32_t count, uint32_t bits) {
  constexpr int kWaves = kBlock / 64;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
  const uint32_t passes = bits > kBucketDigit ? (bits + kBucketDigit - 1) / kBucketDigit : 1, per = (bits + passes - 1) / passes;
  const uint32_t rounds = (count + kBlock - 1) / kBlock, i0 = wave * 64 * rounds + lane;
  uint16_t* off = s.cnt[wave];
#pragma unroll 1
  for (uint32_t pass = 0; pass < passes; ++pass) {
    const uint32_t shift = pass * per, width = min(bits - shift, per), mask = (1u << width) - 1;
    uint32_t rank[kRounds / 2];  // two to a word
    static_assert(kRounds % 2 == 0 && kBucketWords <= 0x10000, "halves of a word");
    uint32_t i = i0;
    __asm__ volatile("" : "+v"(i));  // (else which lanes have an element is kept for all rounds, in more registers than there are)
#pragma unroll
    for (uint32_t b = 0; b < kBucketBins; b += 128) wave_store(reinterpret_cast<uint32_t*>(off + b) + lane, 0u);
    wave_order();
#pragma unroll
    for (uint32_t r = 0; r < kRounds; ++r) {
      if (r % 2 == 0) rank[r / 2] = 0;
      if (r < rounds) {  // block-uniform
        const bool valid = i + r * 64 < count;
        if (pass > 0 && valid) e[r] = room[i + r * 64];
        const uint32_t digit = (sort_key(e[r]) >> shift) & mask;
        const uint64_t peers = same_digit_lanes<kBucketDigit>(digit, valid);
        const uint32_t before = lanes_before(peers);
        const uint32_t there = wave_load(off + digit);
        rank[r / 2] |= (there + before) << (r % 2 * 16);
        wave_order();
        if (valid && before == 0) wave_store(off + digit, (uint16_t)(there + (uint32_t)__popcll(peers)));
        wave_order();
      }
    }
    __syncthreads();  // every wave has counted, and has its elements in registers
    uint32_t c[kWaves], mine = 0;  // a bin per thread
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      c[w] = tid < kBucketBins ? s.cnt[w][tid] : 0u;
      mine += c[w];
    }
    const uint32_t x = wave_sums(mine);
    if (lane == 63) s.wave_sum[wave] = x;
    __syncthreads();
    uint32_t at = x - mine;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kWaves; ++w)
      if (w < wave) at += s.wave_sum[w];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (tid < kBucketBins) s.cnt[w][tid] = (uint16_t)at;
      at += c[w];
    }
    __syncthreads();
    __asm__ volatile("" : "+v"(i));
#pragma unroll
    for (uint32_t r = 0; r < kRounds; ++r)
      if (i + r * 64 < count && r < rounds) room[off[(sort_key(e[r]) >> shift) & mask] + (rank[r / 2] >> (r % 2 * 16) & 0xFFFFu)] = e[r];
    __syncthreads();
  }
}

// A chain of dependent steps in every block, so that what counts is how many blocks run at a time and how few steps there are.
// The pairs are in registers between the digits and in one LDS buffer, so that four blocks fit a compute unit (a million pairs
// have 1024 ordinary bins, all of which run at a time then), and a digit is one walk over them.  With two LDS buffers, two blocks
// to a compute unit and a walk more to count, us: a million pairs 27.4 -> 20.2, 690 K 16.0 -> 13.0, 204 K 11.0 -> 9.5, 26 K 6.0
// either way.  (Blocks of 512 threads spill two registers of a lane for eight waves a SIMD.)
template <int kBlock>
__global__ __launch_bounds__(kBlock, kBlock == 512 ? 8 : 4) void sort_bucket_kernel(Control* __restrict__ ctl, const uint2* __restrict__ src,
                                                             uint32_t items, uint32_t units, uint32_t units_pow2,
                                                             uint32_t buckets_log2, uint32_t group_log2, uint32_t stride,
                                                             const uint32_t* __restrict__ shares,
                                                             const uint32_t* __restrict__ turns_n,
                                                             const uint2* __restrict__ turns, uint2* __restrict__ dst) {
  constexpr int kWaves = kBlock / 64;
  __shared__ BucketLds<kBlock> s;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id(), grid = 1u << buckets_log2;
  const bool ordinary = blockIdx.x < grid;
  // (blocks go round the eight XCDs; neighbouring bins share lines of `shares` and of the units' pairs)
  uint32_t bin = grid < 8 ? blockIdx.x : blockIdx.x % 8 * (grid / 8) + blockIdx.x / 8;
  const auto ask = [&]() { return tid < units ? shares[tid * stride + bin] : 0u; };
  uint32_t share = ordinary ? ask() : 0u;  // (a word that nobody wrote, if the batch has fewer bins)
  const SplitKey split(ctl->hwm, buckets_log2, group_log2);
  const uint32_t hot = (uint32_t)ctl->scratch[kHotBins], inv = split.inverse();
  uint32_t turn = 0;
  if (!ordinary) {
    if (blockIdx.x - grid >= turns_n[0]) return;
    const uint2 w = turns[blockIdx.x - grid];
    bin = w.x;
    turn = w.y;
    share = ask();
  } else if (bin >= split.buckets) {
    return;
  }
  // scans of where the shares begin, whose sum is where the bin does, and of how much they hold
  const uint32_t from = share & 0xFFFFu, len = share >> 16;
  const uint32_t x = wave_sums(from), y = wave_sums(len);
  if (lane == 63) {
    s.wave_sum[wave] = x;
    s.wave_sum[kWaves + wave] = y;
  }
  __syncthreads();
  uint32_t base = 0, count = 0, before = y - len;
#pragma unroll
  for (uint32_t w = 0; w < (uint32_t)kWaves; ++w) {
    base += s.wave_sum[w];
    if (w < wave) before += s.wave_sum[kWaves + w];
    count += s.wave_sum[kWaves + w];
  }
  if (tid < units_pow2) {  // (units past the last one begin behind every pair)
    s.first[tid] = tid < units ? before : 0xFFFFFFFFu;
    s.from[tid] = (uint16_t)from;
  }
  // the last bin ends where all pairs do
  if (bin == split.buckets + hot - 1 && turn >> 16 == 0 && tid == 0)
    ctl->scratch[kValidPairs] = (unsigned long long)base + count;
  __syncthreads();
  if (!ordinary) {  // one row: its pairs are in order
    const uint32_t part = turn >> 16, parts = turn & 0xFFFFu;
    const uint32_t a = (uint32_t)((uint64_t)count * part / parts), e = (uint32_t)((uint64_t)count * (part + 1) / parts);
    for (uint32_t q = a + tid; q < e; q += kBlock * kTogether) {
      uint2 p[kTogether];
      pairs_of_bin(s, units_pow2, items, src, q, kBlock, e, p);
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j)
        if (q + j * kBlock < e) dst[base + q + j * kBlock] = make_uint2(split.row(p[j].x, inv), p[j].y);
    }
    return;
  }
  const uint32_t all = 1u << split.rest, keys = all - 1;
  const uint32_t rounds = (count + kBlock - 1) / kBlock;  // a wave sorts 64 * rounds consecutive pairs
  const uint32_t i0 = wave * 64 * rounds + lane;
  constexpr uint32_t kPairRounds = kBucketMost / kBlock;
  if (count <= kBucketMost) {
    uint2 pair[kPairRounds];
#pragma unroll
    for (uint32_t r = 0; r < kPairRounds; r += kTogether) {
      uint2 p[kTogether] = {};
      if (r < rounds) pairs_of_bin(s, units_pow2, items, src, i0 + r * 64, 64, count, p);
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j) pair[r + j] = p[j];
    }
    sort_bucket(s, pair, s.pairs, count, split.rest);
    for (uint32_t q = tid; q < count; q += kBlock) dst[base + q] = make_uint2(split.row(s.pairs[q].x, inv), s.pairs[q].y);
    return;
  }
  if (count <= kBucketWords && split.rest <= 32 - kPlaceBits) {
    constexpr uint32_t kRounds = kBucketWords / kBlock;
    uint32_t word[kRounds];
#pragma unroll
    for (uint32_t r = 0; r < kRounds; r += kTogether) {
      uint2 p[kTogether] = {};
      if (r < rounds) pairs_of_bin(s, units_pow2, items, src, i0 + r * 64, 64, count, p);
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j) word[r + j] = (p[j].x & keys) << kPlaceBits | ((i0 + (r + j) * 64) & (kBucketWords - 1));
    }
    sort_bucket(s, word, s.words, count, split.rest);
    for (uint32_t q = tid; q < count; q += kBlock * kTogether) {
      uint32_t at[kTogether];
      uint2 p[kTogether];
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j)
        at[j] = q + j * kBlock < count ? s.words[q + j * kBlock] & (kBucketWords - 1) : 0xFFFFFFFEu;
      pairs_at(s, units_pow2, items, src, at, count, p);
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j)
        if (q + j * kBlock < count) dst[base + q + j * kBlock] = make_uint2(split.row(p[j].x, inv), p[j].y);
    }
    return;
  }
  // Ranges [low, high) of the keys within the bucket, one after the other, each with no more pairs than fit into LDS.  A key
  // with more pairs than that is copied.
  uint32_t done = 0, low = 0;
  while (low < all && done < count) {
    uint32_t width = (all - low + kBucketBins - 1) / kBucketBins;  // of a bin of the histogram
    for (;;) {
      if (tid < kBucketBins) s.in_range[tid] = 0;
      __syncthreads();
      for (uint32_t q = tid; q < count; q += kBlock * kTogether) {
        uint2 p[kTogether];
        pairs_of_bin(s, units_pow2, items, src, q, kBlock, count, p);
#pragma unroll
        for (uint32_t j = 0; j < kTogether; ++j) {
          const uint32_t k = p[j].x & keys;
          if (q + j * kBlock < count && k >= low && (k - low) / width < kBucketBins) atomicAdd(&s.in_range[(k - low) / width], 1u);
        }
      }
      __syncthreads();
      // how many of its bins fit together, and the pairs in them
      const uint32_t mine = tid < kBucketBins ? s.in_range[tid] : 0u, sum = wave_sums(mine);
      if (lane == 63) s.wave_sum[wave] = sum;
      if (tid < 2) s.range[tid] = 0;
      if (tid == 0) s.range[2] = mine;
      __syncthreads();
      uint32_t upto = sum;
      for (uint32_t w = 0; w < wave; ++w) upto += s.wave_sum[w];
      if (tid < kBucketBins && upto <= kBucketMost) {
        atomicAdd(&s.range[0], 1u);
        atomicMax(&s.range[1], upto);
      }
      __syncthreads();
      if (s.range[0] || width == 1) break;
      width = (width + kBucketBins - 1) / kBucketBins;  // closer
      __syncthreads();
    }
    const bool copy = s.range[0] == 0;
    const uint32_t high = low + (copy ? 1u : s.range[0] * width), here = copy ? s.range[2] : s.range[1];
    // the range's pairs in order: to LDS, or where they belong
    uint32_t taken = 0;
    for (uint32_t q0 = 0; q0 < count; q0 += kBlock * kTogether) {
      uint2 p[kTogether];
      const uint32_t q = q0 + wave * 64 * kTogether + lane;  // (a wave takes consecutive pairs)
      pairs_of_bin(s, units_pow2, items, src, q, 64, count, p);
      uint64_t m[kTogether];
      uint32_t found = 0;
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j) {
        const uint32_t k = p[j].x & keys;
        m[j] = __ballot(q + j * 64 < count && k >= low && k < high);
        found += (uint32_t)__popcll(m[j]);
      }
      __syncthreads();  // (wave_sum has been read)
      if (lane == 0) s.wave_sum[wave] = found;
      __syncthreads();
      uint32_t at = taken;
#pragma unroll
      for (uint32_t w = 0; w < (uint32_t)kWaves; ++w) {
        if (w < wave) at += s.wave_sum[w];
        taken += s.wave_sum[w];
      }
#pragma unroll
      for (uint32_t j = 0; j < kTogether; ++j) {
        const uint32_t to = at + (uint32_t)__popcll(m[j] & lanes_below());
        if (m[j] >> lane & 1) {
          if (copy)
            dst[base + done + to] = make_uint2(split.row(p[j].x, inv), p[j].y);
          else
            s.pairs[to] = p[j];
        }
        at += (uint32_t)__popcll(m[j]);
      }
    }
    __syncthreads();
    if (!copy) {
      const uint32_t many = (here + kBlock - 1) / kBlock, i = wave * 64 * many + lane;
      uint2 pair[kPairRounds];
#pragma unroll
      for (uint32_t r = 0; r < kPairRounds; ++r) pair[r] = r < many && i + r * 64 < here ? s.pairs[i + r * 64] : make_uint2(0u, 0u);
      sort_bucket(s, pair, s.pairs, here, split.rest);
      for (uint32_t q = tid; q < here; q += kBlock) dst[base + done + q] = make_uint2(split.row(s.pairs[q].x, inv), s.pairs[q].y);
      __syncthreads();
    }
    done += here;
    low = high;
  }
}

template <int kThreads, uint32_t kItems, uint32_t kSamples, uint32_t kBuckets, uint32_t kUnits, bool kSearch>
static void queue_split(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                        const int64_t* d_offsets, uint64_t n_bags, const SplitShape& sh, hipStream_t stream, Profiler* prof) {
  constexpr int kBlock = kUnits <= 256 ? 256 : 512;  // (a thread per unit)
  static_assert(kUnits <= (uint32_t)kBlock, "a thread per unit");
  constexpr uint32_t kHot = kSamples / kSplitHits, kStride = kBuckets + kHot;
  const uint32_t units = (uint32_t)sort_units(n, kItems), most_turns = kHot + (uint32_t)(n / kSplitTurn);
  uint32_t* turns_n = ws.hist + (uint64_t)units * kStride;
  uint2* turns = reinterpret_cast<uint2*>(turns_n + 2);
  uint32_t pow2 = 1;
  while (pow2 < units) pow2 <<= 1;
  MONO_LAUNCH(prof, K_SORT_SPLIT, stream, (sort_split_kernel<kThreads, kItems, kSamples, kBuckets, kSearch>), dim3(units),
              dim3(kThreads), t.ctl, d_rows, (uint32_t)n, d_offsets, n_bags, sh.buckets_log2, sh.group_log2, ws.hist, turns_n,
              turns, ws.pair_a);
  MONO_LAUNCH(prof, K_SORT_BUCKET, stream, sort_bucket_kernel<kBlock>, dim3((1u << sh.buckets_log2) + most_turns),
              dim3(kBlock), t.ctl, ws.pair_a, kItems, units, pow2, sh.buckets_log2, sh.group_log2, kStride, ws.hist, turns_n,
              turns, ws.pair_b);
}

hipError_t launch_split_pairs(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                              const int64_t* d_offsets, uint64_t n_bags, hipStream_t stream, Profiler* prof) {
  const SplitShape sh = split_shape_for(n);
#define MONO_SPLIT(i, search)                                                                   \
  queue_split<kSplitThreads[i], kSplitItems[i], kSplitSamples[i], kSplitBuckets[i],             \
              sort_units(kSplitUpTo[i], kSplitItems[i]), search>(t, ws, d_rows, n, d_offsets, n_bags, sh, stream, prof)
  switch (sh.size) {
    case 0:
      if (split_searches_bags(n, n_bags))
        MONO_SPLIT(0, true);
      else
        MONO_SPLIT(0, false);
      break;
    case 1: MONO_SPLIT(1, false); break;
    case 2: MONO_SPLIT(2, false); break;
    default: MONO_SPLIT(3, false); break;
  }
#undef MONO_SPLIT
  return hipGetLastError();
}

}  // namespace mono
