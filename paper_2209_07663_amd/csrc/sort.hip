// Stable LSD radix sort of (row index, bag) pairs, which brings the occurrences of one embedding row together before the
// gradient reduction: of more pairs than the split takes (sort_split.hip), and, at the end of the file, of so few that one
// block sorts them in LDS.
//
// The key width is decided ON THE DEVICE: row indices are handed out in ascending order, so every
// row in use is below the high-water mark `hwm` kept in the control block.  bit_length(hwm - 1)
// bits are sorted in the fewest passes of equal width that the call's shape allows (kernels.h); the host picks the
// shape and launches the passes that an upper bound of `hwm` needs (it keeps one without waiting for the
// device: see the table's host side) and the superfluous ones return at once.  Pass p reads buffer (p even ? a : b)
// and writes the other one.  Pass 0 reads the row indices as the caller holds them and finds the bag
// of every occurrence from the offsets (no array of bag numbers is ever written to memory); dropped
// occurrences (row -1) are left out by it, and it publishes the number of pairs that remain
// (kValidPairs slot of the control block's scratch).
//
// Unit of work: one block owns kItems consecutive elements, an equal share per wave.  Per pass:
//   hist     per-unit digit histograms (LDS atomics)
//   scan     exclusive scan of every bin along the units, in groups of four; bin totals to `totals`
//   scatter  the block loads its elements into registers (all loads independent); every wave ranks its elements
//            64 at a time by digit matching with ballots (stable: rank = the wave's earlier elements of the digit
//            + lower lanes with it; what the ranking leaves behind are the wave's digit counts, which a loop
//            of LDS atomics counted before: 46 -> 41 us a pass at 5.8 M pairs); the counts become start
//            offsets inside the block, and the elements go IN ORDER into an LDS copy of the block, which is
//            written out with neighbouring threads on neighbouring elements of a bin.  (Scattering
//            straight from the registers sends one 8-byte write per element to the L2: measured, that
//            request rate was what bounded the pass.)
// No kernel spins or waits for another block.
#include "common.h"
#include "kernels.h"
#include "sort_ops.h"

namespace mono {

// A kernel of the sort is compiled for one shape (see kernels.h): kBits = widest digit, kItems = elements owned by a block,
// which has a thread for every bin.
template <uint32_t kBits, uint32_t kItems>
struct Shape {
  static constexpr uint32_t kBins = 1u << kBits;
  static constexpr int kBlock = (int)kBins;
  static constexpr int kWaves = kBlock / 64;
  static constexpr uint32_t kPerWave = kItems / kWaves;
  static constexpr uint32_t kRounds = kPerWave / 64;
  static_assert(kItems % kBins == 0, "whole waves");
};

// The bag that holds occurrence `pos`: the last bag b with offsets[b] <= pos (offsets are non-decreasing
// and start at 0).  Run by a whole wave: 64 probes per step, four dependent steps for two million bags.
// Whatever the offsets hold, the answer is a bag index below n_bags and the loop ends.
__device__ inline uint32_t bag_holding(const int64_t* offsets, uint64_t n_bags, uint64_t n, uint64_t pos) {
  uint64_t lo = 0, hi = n_bags;
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + 63) / 64;
    const uint64_t p = lo + (uint64_t)(lane_id() + 1) * step;
    const bool ok = p < hi && bounded_offset(offsets, p, n) <= pos;
    const uint64_t m = __ballot(ok);
    const uint64_t k = m == ~0ull ? 64 : (uint64_t)(__ffsll((unsigned long long)~m) - 1);  // leading yes answers
    const uint64_t nlo = lo + k * step, nhi = lo + (k + 1) * step;
    lo = nlo;
    hi = nhi < hi ? nhi : hi;
  }
  return (uint32_t)lo;
}

// Threads of a block of sort_hist_kernel.  The wide shape's groups are few: 417 blocks of 6.8 M pairs, whose 13 waves a compute
// unit with 512 threads each left the memory idle (17.7 -> 15.5 us a pass; 43 at 26 M either way).
template <uint32_t kBits>
constexpr int kGroupBlock = kBits > 8 ? 1024 : 512;
constexpr uint32_t kSortChunk = 16;  // see sort_scatter_kernel

// Digit histograms of a group of consecutive units: a unit's words are what the units before it in the group hold, to
// hist[unit * bins + bin]; the group's, to sums[group * bins + bin].  Whole lines are written here and read by the scatter
// kernel, and the scan has kSortGroupUnits times less to read.
// Pass 0 has more blocks than that, in front: for the scatter kernel of the same pass, their waves find the bag that
// holds a unit's first occurrence, a unit each (four dependent memory round trips, beside the counting instead of
// after it).
// LDS atomics to one word cost two cycles each where spread ones take a fifth of a cycle, and a batch has hot rows
// and slots of few IDs: every counter is kept four times, for a quarter of the lanes each.
// Both together: 22.8 -> 12.5 us a pass at 6.8 M pairs in 8-bit digits (reading the pairs takes 10), 75 -> 43 at 26 M
// in 9-bit ones, and 39.6 -> 36.8 and 153 -> 146 in the scatter kernel.  A unit per block instead of four takes 5 us
// less here at 26 M but 11 more in the scan.
template <uint32_t kBits, uint32_t kItems>
__global__ __launch_bounds__(kGroupBlock<kBits>) void sort_hist_kernel(const Control* __restrict__ ctl, uint32_t pass,
                                                               const int32_t* __restrict__ rows,
                                                               const uint2* __restrict__ src, uint64_t n,
                                                               uint32_t* __restrict__ hist,
                                                               uint32_t* __restrict__ sums,
                                                               const int64_t* __restrict__ offsets, uint64_t n_bags,
                                                               uint32_t* __restrict__ unit_bag,
                                                               uint32_t search_blocks) {
  const SortPlan plan = make_sort_plan(ctl->hwm, kBits);
  if (pass >= plan.passes) return;
  constexpr uint32_t kBins = 1u << kBits, kBlock = kGroupBlock<kBits>, kUnits = kSortGroupUnits, kCopies = 4;
  __shared__ uint4 words[kUnits * kBins * kCopies / 4];
  uint32_t* cnt = reinterpret_cast<uint32_t*>(words);  // [unit][bin][copy]
  if (blockIdx.x < search_blocks) {
    const uint64_t unit = (uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (unit * kItems < n) {  // wave-uniform
      const uint32_t b = bag_holding(offsets, n_bags, n, unit * kItems);
      if (lane_id() == 0) unit_bag[unit] = b;
    }
    return;
  }
  const uint64_t block = blockIdx.x - search_blocks;
  const uint32_t shift = plan.shift(pass), nbins = 1u << plan.width(pass), mask = nbins - 1;
  if (pass > 0) n = ctl->scratch[kValidPairs];
  // every key of the thread is requested before the first one is counted (left to itself the compiler
  // keeps each load behind the LDS atomic before it: a memory round trip for each)
  constexpr uint32_t kPerThread = kItems * kUnits / kBlock;
  static_assert(kItems % kBlock == 0, "a round of the block is in one unit");
  uint32_t key[kPerThread];
#pragma unroll
  for (uint32_t r = 0; r < kPerThread; ++r) {
    const uint64_t i = block * kUnits * kItems + (uint64_t)r * kBlock + threadIdx.x;
    key[r] = plan.hwm;
    if (i < n) key[r] = pass == 0 ? first_key(rows, i, plan.hwm) : src[i].x;
  }
  for (uint32_t b = threadIdx.x; b < kUnits * kBins * kCopies / 4; b += kBlock) words[b] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const uint32_t copy = threadIdx.x % kCopies;
#pragma unroll
  for (uint32_t r = 0; r < kPerThread; ++r) {
    const uint32_t bin = r * kBlock / kItems * kBins + ((key[r] >> shift) & mask);
    if (key[r] < plan.hwm) atomicAdd(&cnt[bin * kCopies + copy], 1u);
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < nbins; b += kBlock) {
    uint32_t run = 0;
#pragma unroll
    for (uint32_t u = 0; u < kUnits; ++u) {
      const uint4 c = words[u * kBins + b];
      hist[(block * kUnits + u) * kBins + b] = run;
      run += c.x + c.y + c.z + c.w;
    }
    sums[block * kBins + b] = run;
  }
}

// Exclusive scan of sums[0 .. groups)[bin] in place; total of the bin to totals[bin].  A block owns four bins (16 bytes of
// every group's words); a thread takes consecutive groups, all asked for at once, the threads' sums are scanned
// across the block and the words written back.  Eight blocks share a line: they run on one XCD (blocks go
// round the XCDs), whose L2 then reads and writes the line once.
__device__ inline uint4 plus(uint4 a, uint4 b) { return make_uint4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ inline uint4 minus(uint4 a, uint4 b) { return make_uint4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); }
__device__ inline uint4 wave_scan(uint4 x) {  // inclusive
  return make_uint4(wave_sums(x.x), wave_sums(x.y), wave_sums(x.z), wave_sums(x.w));
}
constexpr int kScanBlock = 1024;
constexpr uint32_t kScanPer = 8;  // groups per thread and round
template <uint32_t kBits>
__global__ __launch_bounds__(kScanBlock) void sort_scan_kernel(const Control* __restrict__ ctl, uint32_t pass,
                                                               uint32_t* __restrict__ sums, uint64_t groups,
                                                               uint32_t* __restrict__ totals) {
  static_assert(kBits >= 8, "whole lines on every XCD");
  const SortPlan plan = make_sort_plan(ctl->hwm, kBits);
  const uint32_t xcd = blockIdx.x % 8, turn = blockIdx.x / 8;                    // the 8 blocks of a line: turns 8 k to 8 k + 7
  const uint32_t strip = (turn / 8 * 8 + xcd) * 8 + turn % 8;
  if (pass >= plan.passes || strip * 4 >= (1u << plan.width(pass))) return;
  constexpr uint32_t kWaves = kScanBlock / 64;
  __shared__ uint4 wave_sum[kWaves];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint4* at = reinterpret_cast<uint4*>(sums) + strip;
  constexpr uint64_t kPitch = (1u << kBits) / 4;
  // (few groups: as few per thread as cover them)
  const uint32_t per = groups >= kScanBlock * kScanPer ? kScanPer : (uint32_t)((groups + kScanBlock - 1) / kScanBlock);
  uint4 carry = make_uint4(0u, 0u, 0u, 0u);
  for (uint64_t u0 = 0; u0 < groups; u0 += (uint64_t)kScanBlock * per) {
    const uint64_t first = u0 + (uint64_t)threadIdx.x * per;
    uint4 v[kScanPer], sum = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
      v[j] = make_uint4(0u, 0u, 0u, 0u);
      if (j < per && first + j < groups) v[j] = at[(first + j) * kPitch];
    }
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) sum = plus(sum, v[j]);
    const uint4 x = wave_scan(sum);
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    uint4 run = plus(carry, minus(x, sum));
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      const uint4 s = wave_sum[w];
      if (w < wave) run = plus(run, s);
      carry = plus(carry, s);
    }
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
      if (j < per && first + j < groups) at[(first + j) * kPitch] = run;
      run = plus(run, v[j]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) reinterpret_cast<uint4*>(totals)[strip] = carry;
}

// kFirst: pass 0 (in a kernel of its own: the code that finds the bags, though skipped, held the loads of the other
// passes together: 26 M pairs 133 -> 113 and 107 -> 92 us a pass)
template <uint32_t kBits, uint32_t kItems, bool kFirst>
__global__ __launch_bounds__(1 << kBits) void sort_scatter_kernel(Control* __restrict__ ctl, uint32_t pass,
                                                                  const int32_t* __restrict__ rows,
                                                                  const int64_t* __restrict__ offsets,
                                                                  uint64_t n_bags, const uint32_t* __restrict__ unit_bag,
                                                                  const uint2* __restrict__ src,
                                                                  uint64_t n, const uint32_t* __restrict__ hist,
                                                                  const uint32_t* __restrict__ sums,
                                                                  const uint32_t* __restrict__ totals,
                                                                  uint2* __restrict__ dst) {
  const SortPlan plan = make_sort_plan(ctl->hwm, kBits);
  if (pass >= plan.passes) return;
  // The large blocks serve batches whose pairs do not stay in the 256 MB cache behind the L2s until the next pass: read
  // past it they leave room for the pairs being written (a pass over 26 M pairs 170 -> 153 us; over 6.8 M the same)
  constexpr bool kLoadOnce = kItems >= 4096;
  using S = Shape<kBits, kItems>;
  constexpr int kBlock = S::kBlock;
  __shared__ uint2 stage[kItems];          // the block's elements in sorted order
  __shared__ uint32_t lds[S::kWaves][S::kBins];   // per-wave digit counts, then local start offsets
  __shared__ uint32_t local_start[S::kBins];       // first position of a bin in `stage`
  __shared__ uint32_t global_start[S::kBins];      // where this block's part of a bin goes in dst
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t* bag_here = reinterpret_cast<uint32_t*>(stage);  // (pass 0, until step 4)
  // Which unit: blocks go round the eight XCDs, and the elements that neighbouring units have of a bin share lines, so
  // that an XCD takes kSortChunk neighbouring units and its L2 writes whole lines (26 M pairs: 187 -> 161,
  // 114 -> 103 and 92 -> 91 us; chunks of 4, 64 or an eighth of the batch are a few us behind).
  const uint32_t turn = blockIdx.x / 8;
  const uint64_t unit = ((uint64_t)(turn / kSortChunk) * 8 + blockIdx.x % 8) * kSortChunk + turn % kSortChunk;
  if (unit * kItems >= n) return;  // (the grid is a whole number of chunks)
  const uint32_t last_bag = (uint32_t)(n_bags - 1);
  const uint32_t shift = plan.shift(pass), nbins = 1u << plan.width(pass), mask = nbins - 1;

  // 0. what step 3 needs from memory is asked for first: it arrives while the elements are loaded
  const uint32_t bin = threadIdx.x;  // the thread's bin
  uint32_t tot = 0, before_me = 0;   // its pairs in the whole batch / in the units before this one
  if (bin < nbins) {
    tot = totals[bin];
    before_me = hist[unit * S::kBins + bin] + sums[unit / kSortGroupUnits * S::kBins + bin];
  }
  // 1. this wave's elements -> registers (independent, coalesced loads)
  if constexpr (!kFirst) n = ctl->scratch[kValidPairs];
  const uint64_t ubase = unit * kItems;
  const uint64_t base = ubase + (uint64_t)wave * S::kPerWave;
  uint2 kv[S::kRounds];
#pragma unroll
  for (uint32_t r = 0; r < S::kRounds; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    kv[r] = make_uint2(0xFFFFFFFFu, 0u);
    if (i < n) {
      if constexpr (kFirst)
        kv[r] = make_uint2(first_key(rows, i, plan.hwm), 0u);
      else
        kv[r] = kLoadOnce ? load_once(src + i) : src[i];
    }
    if (kv[r].x >= plan.hwm) kv[r].x = 0xFFFFFFFFu;  // dropped occurrence (or past the end): left out
  }
  // (pass 0) the unit's bags from the one that holds its first occurrence on, neighbouring threads
  // neighbouring bags; the first of them start to arrive during step 2
  constexpr uint32_t kBagsAhead = 2;
  const uint64_t uend = ubase + kItems < n ? ubase + kItems : n;
  uint64_t bag = 0;
  uint32_t start[kBagsAhead];
  const auto ask = [&]() {
#pragma unroll
    for (uint32_t q = 0; q < kBagsAhead; ++q) {
      const uint64_t b = bag + q * kBlock;
      start[q] = (uint32_t)(b < n_bags ? bounded_offset(offsets, b, n) : uend);
    }
  };
  if constexpr (kFirst) {
    bag = (uint64_t)unit_bag[unit] + threadIdx.x;
    ask();
    for (uint32_t p = threadIdx.x; p < kItems; p += kBlock) bag_here[p] = 0;
  }
  for (uint32_t b = threadIdx.x; b < S::kBins; b += kBlock) {
#pragma unroll
    for (int w = 0; w < S::kWaves; ++w) lds[w][b] = 0;
  }
  __syncthreads();
  // 2. rank of every element among the wave's elements of its digit (stable), 64 at a time; what is left in
  //    `lds` is the wave's digit counts
  uint32_t rank[S::kRounds];  // digit << 16 | rank
  {
    uint32_t* off = lds[wave];
#pragma unroll
    for (uint32_t r = 0; r < S::kRounds; ++r) {
      const bool valid = kv[r].x != 0xFFFFFFFFu;
      const uint32_t digit = (kv[r].x >> shift) & mask;
      const uint64_t peers = same_digit_lanes<kBits>(digit, valid);
      const uint32_t before = lanes_before(peers);
      rank[r] = (digit << 16) | (wave_load(off + digit) + before);
      wave_order();
      if (valid && before == 0) wave_store(off + digit, (rank[r] & 0xFFFFu) + (uint32_t)__popcll(peers));
      wave_order();
    }
  }
  static_assert(kItems <= 0x10000, "rank and digit share a word");
  __syncthreads();
  // 3. exclusive scans of the bins' counts, once within the block (positions in `stage`) and once over all bins of the
  //    pass (start of the bin in dst)
  __shared__ uint32_t scan_sum[S::kWaves], scan_tot[S::kWaves];
  {
    uint32_t mine = 0;
#pragma unroll
    for (int w = 0; w < S::kWaves; ++w) mine += lds[w][bin];
    const uint32_t x = wave_sums(mine), y = wave_sums(tot);
    if (lane == 63) {
      scan_sum[wave] = x;
      scan_tot[wave] = y;
    }
    __syncthreads();
    uint32_t run = x - mine, run_tot = y - tot;  // first position of the bin in the block / in dst
#pragma unroll 1  // (unrolled it holds registers that cost the wide shape a wave in six)
    for (uint32_t w = 0; w < wave; ++w) {
      run += scan_sum[w];
      run_tot += scan_tot[w];
    }
    local_start[bin] = run;
    global_start[bin] = run_tot + before_me;
#pragma unroll
    for (int w = 0; w < S::kWaves; ++w) {
      const uint32_t c = lds[w][bin];
      lds[w][bin] = run;
      run += c;
    }
    if (kFirst && unit == 0 && bin == S::kBins - 1) ctl->scratch[kValidPairs] = run_tot + tot;  // pairs that remain
  }
  if constexpr (kFirst) {
    // The bag of every occurrence of the unit (the pooled gradient of bag b is the gradient of each of its
    // occurrences): every bag leaves its number at its first occurrence (of bags that start at one place the last is
    // the one that is not empty), and an occurrence takes the number left at or before it.  Offsets are
    // non-decreasing: a thread stops at its first bag that starts at or after the end of the unit.  Whatever they
    // hold, every write stays inside the unit and every bag number that is used is bounded to the bags of the batch.
    __shared__ uint32_t wave_last[S::kWaves];
    for (bool more = true; more;) {
#pragma unroll
      for (uint32_t q = 0; q < kBagsAhead; ++q) {
        const uint64_t b = bag + q * kBlock;
        const uint64_t at = start[q] > ubase ? start[q] - ubase : 0;
        more = b < n_bags && start[q] < uend;
        if (more) atomicMax(&bag_here[at], (uint32_t)b + 1u);
      }
      bag += (uint64_t)kBlock * kBagsAhead;
      if (more) ask();
    }
    __syncthreads();
    uint32_t carry = 0;  // the last number left in the wave's earlier elements
#pragma unroll
    for (uint32_t r = 0; r < S::kRounds; ++r) {
      const uint32_t mark = bag_here[wave * S::kPerWave + r * 64 + lane];
      kv[r].y = max(wave_maxima(mark), carry);
      carry = lane_value(kv[r].y, 63);
    }
    if (lane == 0) wave_last[wave] = carry;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before = wave_last[w] ? wave_last[w] : before;
#pragma unroll
    for (uint32_t r = 0; r < S::kRounds; ++r) {
      const uint32_t b = kv[r].y ? kv[r].y : before;
      kv[r].y = min(b ? b - 1u : 0u, last_bag);
    }
  }
  __syncthreads();
  // 4. into `stage`, in sorted order
#pragma unroll
  for (uint32_t r = 0; r < S::kRounds; ++r)
    if (kv[r].x != 0xFFFFFFFFu) stage[lds[wave][rank[r] >> 16] + (rank[r] & 0xFFFFu)] = kv[r];
  __syncthreads();
  // 5. out: neighbouring threads write neighbouring elements of a bin
  uint32_t total = 0;
#pragma unroll
  for (int w = 0; w < S::kWaves; ++w) total += scan_sum[w];
  for (uint32_t p = threadIdx.x; p < total; p += kBlock) {
    const uint2 e = stage[p];
    const uint32_t digit = (e.x >> shift) & mask;
    dst[global_start[digit] + (p - local_start[digit])] = e;
  }
}

// The whole sort of a batch of at most kSortSmall pairs by one block, all passes in LDS, in one launch.
constexpr int kSmallBlock = 1024;
constexpr uint32_t kSmallWaves = kSmallBlock / 64, kSmallRounds = (uint32_t)kSortSmall / kSmallBlock;
constexpr uint32_t kSmallBag = 32, kSmallLong = (uint32_t)kSortSmall / kSmallBag;  // a longer bag is a long one; room for all of them
__global__ __launch_bounds__(kSmallBlock) void sort_small_kernel(Control* __restrict__ ctl, const int32_t* __restrict__ rows,
                                                                 uint32_t n, const int64_t* __restrict__ offsets,
                                                                 uint64_t n_bags, uint2* __restrict__ dst) {
  constexpr uint32_t kBins = 1u << kSortNarrowBits;
  const SortPlan plan = make_sort_plan(ctl->hwm, kSortNarrowBits);
  __shared__ uint2 pairs[kSortSmall];
  __shared__ uint32_t cnt[kSmallWaves][kBins];
  __shared__ uint32_t wave_sum[kBins / 64];
  __shared__ uint4 long_bag[kSmallLong];  // bag, first and last of the occurrences that it has not written yet
  __shared__ uint32_t n_long;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
  const uint32_t rounds = (n + kSmallBlock - 1) / kSmallBlock;  // a wave owns 64 * rounds consecutive pairs
  const uint32_t i0 = wave * 64 * rounds + lane;
  uint2 kv[kSmallRounds];
#pragma unroll
  for (uint32_t r = 0; r < kSmallRounds; ++r) {
    const uint32_t i = i0 + r * 64;
    kv[r] = make_uint2(0xFFFFFFFFu, 0u);
    if (r < rounds && i < n) kv[r].x = first_key(rows, i, plan.hwm);
    if (kv[r].x >= plan.hwm) kv[r].x = 0xFFFFFFFFu;  // dropped occurrence (or past the end): left out
  }
  {  // every bag writes its number over its occurrences (all bags: a small batch has few), a long one by a whole wave
    // (by its thread alone, the only bag of 8192 pairs made the update take 294 us, 35 so)
    uint32_t* bag_here = reinterpret_cast<uint32_t*>(pairs);
    if (tid == 0) n_long = 0;
    __syncthreads();
    for (uint64_t b = tid; b < n_bags; b += kSmallBlock) {
      const uint32_t from = (uint32_t)bounded_offset(offsets, b, n), to = (uint32_t)bounded_offset(offsets, b + 1, n);
      const uint32_t end = to > from && to - from > kSmallBag ? from + kSmallBag : to;
      for (uint32_t i = from; i < end; ++i) bag_here[i] = (uint32_t)b;
      if (end < to) {
        const uint32_t at = atomicAdd(&n_long, 1u);
        if (at < kSmallLong) long_bag[at] = make_uint4((uint32_t)b, end, to, 0u);  // (else the offsets decrease somewhere)
      }
    }
    __syncthreads();
    const uint32_t longs = n_long < kSmallLong ? n_long : kSmallLong;
    if (longs) {  // block-uniform
      for (uint32_t q = wave; q < longs; q += kSmallWaves) {
        const uint4 x = long_bag[q];
        for (uint32_t i = x.y + lane; i < x.z; i += 64) bag_here[i] = x.x;
      }
      __syncthreads();
    }
    const uint32_t last_bag = (uint32_t)(n_bags - 1);  // (an occurrence outside every bag reads whatever the LDS held)
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; ++r)
      if (r < rounds) kv[r].y = min(bag_here[i0 + r * 64], last_bag);
  }
  uint32_t count = n;  // elements that the pass reads: all occurrences, then the pairs that remain
#pragma unroll 1
  for (uint32_t pass = 0; pass < plan.passes; ++pass) {
    const uint32_t shift = plan.shift(pass), mask = (1u << plan.width(pass)) - 1;
    if (pass > 0) {
#pragma unroll
      for (uint32_t r = 0; r < kSmallRounds; ++r)
        kv[r] = r < rounds && i0 + r * 64 < count ? pairs[i0 + r * 64] : make_uint2(0xFFFFFFFFu, 0u);
    }
    uint32_t* off = cnt[wave];
#pragma unroll
    for (uint32_t b = 0; b < kBins; b += 64) wave_store(off + b + lane, 0u);
    wave_order();
    uint32_t rank[kSmallRounds];  // digit << 16 | rank among the wave's elements of the digit
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; ++r) {
      rank[r] = 0;
      if (r < rounds) {  // block-uniform
        const bool valid = kv[r].x != 0xFFFFFFFFu;
        const uint32_t digit = (kv[r].x >> shift) & mask;
        const uint64_t peers = same_digit_lanes<kSortNarrowBits>(digit, valid);
        const uint32_t before = lanes_before(peers);
        rank[r] = (digit << 16) | (wave_load(off + digit) + before);
        wave_order();
        if (valid && before == 0) wave_store(off + digit, (rank[r] & 0xFFFFu) + (uint32_t)__popcll(peers));
        wave_order();
      }
    }
    __syncthreads();  // every wave has counted, and has its pairs in registers
    uint32_t mine = 0;
    if (tid < kBins) {
#pragma unroll
      for (uint32_t w = 0; w < kSmallWaves; ++w) mine += cnt[w][tid];
    }
    const uint32_t x = wave_sums(mine);
    if (tid < kBins && lane == 63) wave_sum[wave] = x;
    __syncthreads();
    if (tid < kBins) {
      uint32_t at = x - mine;
      for (uint32_t w = 0; w < wave; ++w) at += wave_sum[w];
#pragma unroll
      for (uint32_t w = 0; w < kSmallWaves; ++w) {
        const uint32_t c = cnt[w][tid];
        cnt[w][tid] = at;
        at += c;
      }
    }
    count = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; ++r)
      if (kv[r].x != 0xFFFFFFFFu) pairs[cnt[wave][rank[r] >> 16] + (rank[r] & 0xFFFFu)] = kv[r];
    __syncthreads();
  }
  for (uint32_t i = tid; i < count; i += kSmallBlock) dst[i] = pairs[i];
  if (tid == 0) ctl->scratch[kValidPairs] = count;
}

hipError_t launch_sort_small(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                             const int64_t* d_offsets, uint64_t n_bags, hipStream_t stream, Profiler* prof) {
  MONO_LAUNCH(prof, K_SORT_SCATTER, stream, sort_small_kernel, dim3(1), dim3(kSmallBlock), t.ctl, d_rows, (uint32_t)n, d_offsets,
              n_bags, ws.pair_b);
  return hipGetLastError();
}

template <uint32_t kBits, uint32_t kItems>
static void queue_sort_passes(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                              const int64_t* d_offsets, uint64_t n_bags, uint32_t passes, hipStream_t stream,
                              Profiler* prof) {
  const uint64_t units = sort_units(n, kItems), groups = sort_groups(n, kItems);
  uint32_t* sums = ws.hist + ((groups * kSortGroupUnits) << kBits);
  uint32_t* totals = sums + (groups << kBits);
  const uint64_t chunks = 8 * kSortChunk;  // whole chunks on every XCD
  const dim3 block(Shape<kBits, kItems>::kBlock), grid((unsigned)((units + chunks - 1) / chunks * chunks));
  for (uint32_t p = 0; p < passes; ++p) {
    const uint2* src = p % 2 == 0 ? ws.pair_a : ws.pair_b;
    uint2* dst = p % 2 == 0 ? ws.pair_b : ws.pair_a;
    const uint32_t search = p == 0 ? (uint32_t)((units + kGroupBlock<kBits> / 64 - 1) / (kGroupBlock<kBits> / 64)) : 0u;
    MONO_LAUNCH(prof, K_SORT_HIST, stream, (sort_hist_kernel<kBits, kItems>), dim3((unsigned)groups + search), dim3(kGroupBlock<kBits>),
                t.ctl, p, d_rows, src, n, ws.hist, sums, d_offsets, n_bags, ws.unit_bag, search);
    MONO_LAUNCH(prof, K_SORT_SCAN, stream, sort_scan_kernel<kBits>, dim3((1u << kBits) / 4), dim3(kScanBlock), t.ctl, p, sums,
                groups, totals);
    if (p == 0)
      MONO_LAUNCH(prof, K_SORT_SCATTER, stream, (sort_scatter_kernel<kBits, kItems, true>), grid, block, t.ctl, p, d_rows,
                  d_offsets, n_bags, ws.unit_bag, src, n, ws.hist, sums, totals, dst);
    else
      MONO_LAUNCH(prof, K_SORT_SCATTER, stream, (sort_scatter_kernel<kBits, kItems, false>), grid, block, t.ctl, p, d_rows,
                  d_offsets, n_bags, ws.unit_bag, src, n, ws.hist, sums, totals, dst);
  }
}

hipError_t launch_sort_pairs(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                             const int64_t* d_offsets, uint64_t n_bags, uint32_t hwm_bound, uint32_t* launched,
                             uint32_t* max_bits, hipStream_t stream, Profiler* prof) {
  // the shape and as many passes as the largest high-water mark the table can have by now needs (the device
  // knows the real mark: passes beyond its plan return at once)
  const uint32_t bound = hwm_bound < (uint32_t)t.capacity ? hwm_bound : (uint32_t)t.capacity;
  const SortShape shape = sort_shape_for(bound);
  const SortPlan worst = make_sort_plan(bound, shape.max_bits);
  *launched = worst.passes;
  *max_bits = shape.max_bits;
  if (shape.max_bits == kSortWideBits)
    queue_sort_passes<kSortWideBits, kSortWideItems>(t, ws, d_rows, n, d_offsets, n_bags, worst.passes, stream, prof);
  else
    queue_sort_passes<kSortNarrowBits, kSortNarrowItems>(t, ws, d_rows, n, d_offsets, n_bags, worst.passes, stream, prof);
  return hipGetLastError();
}

}  // namespace mono
