// Brings exported elements into ascending order of their keys (as unsigned numbers) on the device.
//
// A snapshot or a delta is compared, merged and sent in key order; sorting 42 K exported keys and picking their
// rows in that order on the host took 3 ms of a 6.3 ms synchronisation step.
//
// Keys of a table are distinct, and a key's place is the number of smaller ones.  Small exports are put in order by counting:
//   up to kRankMost    `rank`: sixteen lanes compare a key with all others, which lie in LDS, and it is written where it belongs
//   up to kRangesMost  `rank` puts a sample in order, every eighth key of which begins a range of about 256 keys; `ranges`: a
//                      block per range reads all keys, counts those before the range, collects the range's in LDS and ranks them
// One launch and two, where the passes below are three for every eight bits: 42 K keys of a 2^40 space 51 -> 22 us; deltas of
// 125 to 17 K keys, whole calls, 200-250 -> 115-165 us.
// Larger ones by a stable LSD radix sort of (key, index) pairs, eight bits a pass, over the bits in which the keys differ at all
// (IDs of a 2^40 space: five passes).  Per pass:
//   hist     digit histogram of every unit of elements, bin-major
//   scan     one block per bin: exclusive scan along the units, total of the bin
//   scatter  a block ranks its unit (stable, by ballot matching within a wave) into LDS and writes it out
// Then `emit` writes keys and attributes in order; the rows follow through the ordinary export_values kernel.
// Exports of some 100 K keys are bound by the latency of these launches, large ones by the 24 bytes that a pass moves per
// element.
#include "common.h"
#include "kernels.h"
#include "sort_ops.h"

namespace mono {

constexpr int kThreads = 256, kWaves = kThreads / 64;
// Elements per block: many, so that a bin's share leaves in long pieces, or few where the export is small and a pass
// is the latency of one block.
constexpr uint32_t kUnitLarge = 2048, kUnitSmall = 512;
constexpr uint64_t kSmallExport = 400000;

uint64_t export_sort_units(uint64_t n) {
  const uint64_t large = (n + kUnitLarge - 1) / kUnitLarge, m = n < kSmallExport ? n : kSmallExport;
  const uint64_t small = (m + kUnitSmall - 1) / kUnitSmall;
  return large > small ? large : small;
}

constexpr uint32_t kRankMost = 4096, kRankLanes = 16, kOversample = 8, kMostRanges = 256, kRangeKeys = 256;

struct ExportOut {
  int64_t* keys;
  int32_t* rows;
  uint32_t* last_seen;  // may be null
  int64_t* slot;        // may be null
};
__device__ inline void emit(const ExportWorkspace& ws, const ExportOut& out, uint64_t to, uint64_t key, uint32_t from) {
  out.keys[to] = (int64_t)key;
  out.rows[to] = ws.row[from];
  if (out.last_seen) out.last_seen[to] = ws.seen[from];
  if (out.slot) out.slot[to] = ws.slot[from];
}

// The rank of each of n keys, the ones at i * stride, i < n, of the export's.  bounds == nullptr: all keys (stride == 1), each
// goes where it belongs; else every kOversample-th key, in order, to `bounds`.  Bound by the comparisons: 16 lanes a
// key, so that 4096 keys are 256 blocks and 256 comparisons a lane.
__global__ __launch_bounds__(kThreads) void export_rank_kernel(ExportWorkspace ws, uint32_t stride, uint32_t n, ExportOut out,
                                                               uint64_t* __restrict__ bounds) {
  __shared__ uint64_t s_key[kRankMost];
#pragma unroll 8
  for (uint32_t i = threadIdx.x; i < n; i += kThreads) s_key[i] = ws.key[0][i * stride];
  __syncthreads();
  const uint32_t i = blockIdx.x * (kThreads / kRankLanes) + threadIdx.x / kRankLanes;
  const uint64_t key = i < n ? s_key[i] : 0;
  uint32_t rank = 0;
#pragma unroll 8
  for (uint32_t j = threadIdx.x % kRankLanes; j < n; j += kRankLanes) rank += s_key[j] < key ? 1u : 0u;
  rank = (uint32_t)group_sum((float)rank, kRankLanes);  // (whole numbers below 2^24: exact)
  if (i >= n || threadIdx.x % kRankLanes != 0) return;
  if (!bounds)
    emit(ws, out, rank, key, i);
  else if (rank % kOversample == 0)
    bounds[rank / kOversample] = key;
}

// Range r holds the keys from bounds[r] on (the first: all) that are below bounds[r + 1] (the last: all).  A block reads all
// keys from the L2, bound by the latency of that: sixteen waves, eight keys of a lane in flight (42 K keys, 256 blocks: 16 us,
// with four waves 31).
constexpr int kRangeThreads = 1024;
__global__ __launch_bounds__(kRangeThreads) void export_ranges_kernel(ExportWorkspace ws, uint32_t n, uint32_t ranges,
                                                                 const uint64_t* __restrict__ bounds, ExportOut out) {
  constexpr uint32_t kRoom = 2048;
  __shared__ uint64_t s_key[kRoom];
  __shared__ uint32_t s_from[kRoom], s_count, s_below;
  uint64_t low = blockIdx.x == 0 ? 0 : bounds[blockIdx.x];
  const bool last = blockIdx.x == ranges - 1;
  const uint64_t end = last ? ~0ull : bounds[blockIdx.x + 1];  // (~0 is no key)
  uint64_t high = end;
  // Once, unless a range holds more keys than there is room for, eight times what a range of 64 K keys should and four times
  // of 128 K: it is halved then, for as long as that takes.
  while (low < end) {
    if (threadIdx.x == 0) s_count = s_below = 0;
    __syncthreads();
    uint32_t below = 0;
    constexpr uint32_t kAhead = 8;
    for (uint32_t i0 = 0; i0 < n; i0 += kRangeThreads * kAhead) {
      uint64_t k[kAhead];
#pragma unroll
      for (uint32_t q = 0; q < kAhead; ++q) {
        const uint32_t i = i0 + q * kRangeThreads + threadIdx.x;
        k[q] = i < n ? ws.key[0][i] : ~0ull;
      }
#pragma unroll
      for (uint32_t q = 0; q < kAhead; ++q) {
        below += k[q] < low ? 1u : 0u;
        if (k[q] >= low && k[q] < high) {
          const uint32_t at = atomicAdd(&s_count, 1u);
          if (at < kRoom) {
            s_key[at] = k[q];
            s_from[at] = i0 + q * kRangeThreads + threadIdx.x;
          }
        }
      }
    }
    below = (uint32_t)group_sum((float)below, 64);  // (exact: a wave reads fewer than 2^24 keys)
    if (lane_id() == 0) atomicAdd(&s_below, below);
    __syncthreads();
    const uint32_t count = s_count, before = s_below;
    if (count > kRoom) {  // block-uniform
      high = low + (high - low) / 2;  // (the keys are distinct: at least two of them, so that both halves are real)
      __syncthreads();
      continue;
    }
    constexpr uint32_t kLanes = 4;  // to a key
    const uint32_t part = threadIdx.x % kLanes;
    for (uint32_t i0 = 0; i0 < count; i0 += kRangeThreads / kLanes) {  // block-uniform
      const uint32_t i = i0 + threadIdx.x / kLanes;
      const uint64_t key = i < count ? s_key[i] : 0;
      uint32_t rank = 0;
#pragma unroll 8
      for (uint32_t j = part; j < count; j += kLanes) rank += s_key[j] < key ? 1u : 0u;
      rank = (uint32_t)group_sum((float)rank, kLanes);
      if (i < count && part == 0) emit(ws, out, before + rank, key, s_from[i]);
    }
    __syncthreads();
    low = high;
    high = end;
  }
}

// OR and AND of the keys that the scan has found (at most max_n were written)
__global__ __launch_bounds__(kThreads) void export_bits_kernel(const uint64_t* __restrict__ keys, uint64_t max_n,
                                                               Control* __restrict__ ctl) {
  __shared__ unsigned long long s_any[kWaves], s_all[kWaves];
  const unsigned long long found = ctl->scratch[kExportCount];
  const uint64_t n = found < max_n ? found : max_n;
  unsigned long long any = 0, all = ~0ull;
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kThreads) {
    any |= keys[i];
    all &= keys[i];
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    any |= __shfl_xor(any, d);
    all &= __shfl_xor(all, d);
  }
  if (lane_id() == 0) {
    s_any[threadIdx.x >> 6] = any;
    s_all[threadIdx.x >> 6] = all;
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // (one pair of atomics per block: they serialise)
    for (int w = 1; w < kWaves; ++w) {
      any |= s_any[w];
      all &= s_all[w];
    }
    atomicOr(&ctl->scratch[kExportBits], any);
    atomicAnd(&ctl->scratch[kExportBits + 1], all);
  }
}

template <uint32_t kUnit>
__global__ __launch_bounds__(kThreads) void export_hist_kernel(const uint64_t* __restrict__ keys, uint64_t n,
                                                               uint32_t shift, uint64_t units,
                                                               uint32_t* __restrict__ hist) {
  __shared__ uint32_t cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = (uint64_t)blockIdx.x * kUnit;
#pragma unroll
  for (uint32_t r = 0; r < kUnit / kThreads; ++r) {
    const uint64_t i = base + (uint64_t)r * kThreads + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(uint64_t)threadIdx.x * units + blockIdx.x] = cnt[threadIdx.x];
}

// exclusive scan of one bin's counts along the units, in place; total of the bin to totals[bin]
__global__ __launch_bounds__(kThreads) void export_scan_kernel(uint32_t* __restrict__ hist, uint64_t units,
                                                               uint32_t* __restrict__ totals) {
  __shared__ uint32_t wave_sum[kWaves];
  uint32_t* row = hist + (uint64_t)blockIdx.x * units;
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (uint64_t u0 = 0; u0 < units; u0 += kThreads) {
    const uint64_t u = u0 + threadIdx.x;
    const uint32_t v = u < units ? row[u] : 0u;
    const uint32_t x = wave_sums(v);
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    uint32_t before = carry, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      if (w < wave) before += wave_sum[w];
      all += wave_sum[w];
    }
    if (u < units) row[u] = before + x - v;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// src_idx == nullptr: first pass, an element's index is its position
template <uint32_t kUnit>
__global__ __launch_bounds__(kThreads) void export_scatter_kernel(const uint64_t* __restrict__ src_key,
                                                                  const uint32_t* __restrict__ src_idx, uint64_t n,
                                                                  uint32_t shift, uint64_t units,
                                                                  const uint32_t* __restrict__ hist,
                                                                  const uint32_t* __restrict__ totals,
                                                                  uint64_t* __restrict__ dst_key,
                                                                  uint32_t* __restrict__ dst_idx) {
  constexpr uint32_t kRounds = kUnit / kThreads;  // elements per lane of a wave
  __shared__ uint64_t s_key[kUnit];
  __shared__ uint32_t s_idx[kUnit];
  __shared__ uint32_t cnt[kWaves][256];  // per-wave digit counts, then local start offsets
  __shared__ uint32_t local_start[256], global_start[256], sum_w[kWaves], tot_w[kWaves];
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const uint32_t tot = totals[tid], before_me = hist[(uint64_t)tid * units + blockIdx.x];  // thread <-> bin
#pragma unroll
  for (int w = 0; w < kWaves; ++w) cnt[w][tid] = 0;
  const uint64_t base = (uint64_t)blockIdx.x * kUnit + (uint64_t)wave * (kUnit / kWaves);
  uint64_t key[kRounds];
  uint32_t idx[kRounds];
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    key[r] = i < n ? src_key[i] : 0;
    idx[r] = i < n ? (src_idx ? src_idx[i] : (uint32_t)i) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r)
    if (base + (uint64_t)r * 64 + lane < n) atomicAdd(&cnt[wave][(key[r] >> shift) & 255u], 1u);
  __syncthreads();
  uint32_t mine = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mine += cnt[w][tid];
  const uint32_t x = wave_sums(mine), y = wave_sums(tot);
  if (lane == 63) {
    sum_w[wave] = x;
    tot_w[wave] = y;
  }
  __syncthreads();
  uint32_t at = x - mine, all = y - tot;
  for (uint32_t w = 0; w < wave; ++w) {
    at += sum_w[w];
    all += tot_w[w];
  }
  local_start[tid] = at;
  global_start[tid] = all + before_me;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t c = cnt[w][tid];
    cnt[w][tid] = at;
    at += c;
  }
  __syncthreads();
  uint32_t* off = cnt[wave];
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    const bool valid = base + (uint64_t)r * 64 + lane < n;
    const uint32_t digit = (uint32_t)(key[r] >> shift) & 255u;
    const uint64_t peers = same_digit_lanes<8>(digit, valid);
    const uint32_t before = lanes_before(peers), at = wave_load(off + digit);
    if (valid) {
      s_key[at + before] = key[r];
      s_idx[at + before] = idx[r];
    }
    wave_order();
    if (valid && before == 0) wave_store(off + digit, at + (uint32_t)__popcll(peers));
    wave_order();
  }
  __syncthreads();
  const uint64_t ubase = (uint64_t)blockIdx.x * kUnit;
  const uint32_t here = (uint32_t)(n - ubase < kUnit ? n - ubase : kUnit);
  for (uint32_t p = tid; p < here; p += kThreads) {
    const uint64_t kk = s_key[p];
    const uint32_t digit = (uint32_t)(kk >> shift) & 255u;
    const uint64_t to = (uint64_t)global_start[digit] + (p - local_start[digit]);
    dst_key[to] = kk;
    dst_idx[to] = s_idx[p];
  }
}

__global__ __launch_bounds__(kThreads) void export_emit_kernel(ExportWorkspace ws, const uint64_t* __restrict__ key,
                                                               const uint32_t* __restrict__ idx, uint64_t n, ExportOut out) {
  const uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) emit(ws, out, i, key[i], idx ? idx[i] : (uint32_t)i);
}

hipError_t launch_export_bits(const TableView& t, const ExportWorkspace& ws, uint64_t max_n, hipStream_t stream) {
  const uint64_t blocks = (max_n + kThreads - 1) / kThreads;
  hipLaunchKernelGGL(export_bits_kernel, dim3((unsigned)(blocks < 64 ? (blocks ? blocks : 1) : 64)), dim3(kThreads), 0, stream,
                     ws.key[0], max_n, t.ctl);
  return hipGetLastError();
}

template <uint32_t kUnit>
static hipError_t queue_export_sort(const ExportWorkspace& ws, uint64_t n, uint64_t varying, const ExportOut& out,
                                    hipStream_t stream) {
  const uint64_t units = (n + kUnit - 1) / kUnit;
  uint32_t* totals = ws.hist + 256 * units;
  const dim3 block(kThreads), grid((unsigned)units);
  int side = 0;
  const uint32_t* idx = nullptr;
  for (uint32_t shift = varying ? (uint32_t)__builtin_ctzll(varying) : 64; shift < 64 && (varying >> shift); shift += 8) {
    hipLaunchKernelGGL(export_hist_kernel<kUnit>, grid, block, 0, stream, ws.key[side], n, shift, units, ws.hist);
    hipLaunchKernelGGL(export_scan_kernel, dim3(256), block, 0, stream, ws.hist, units, totals);
    hipLaunchKernelGGL(export_scatter_kernel<kUnit>, grid, block, 0, stream, ws.key[side], idx, n, shift, units, ws.hist,
                       totals, ws.key[1 - side], ws.idx[1 - side]);
    side = 1 - side;
    idx = ws.idx[side];
  }
  hipLaunchKernelGGL(export_emit_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), block, 0, stream, ws,
                     ws.key[side], idx, n, out);
  return hipGetLastError();
}

hipError_t launch_export_sort(const ExportWorkspace& ws, uint64_t n, uint64_t varying, int64_t* d_keys, int32_t* d_row,
                              uint32_t* d_last_seen, int64_t* d_slot, hipStream_t stream) {
  const ExportOut out = {d_keys, d_row, d_last_seen, d_slot};
  if (n > kRangesMost)
    return n <= kSmallExport ? queue_export_sort<kUnitSmall>(ws, n, varying, out, stream)
                             : queue_export_sort<kUnitLarge>(ws, n, varying, out, stream);
  uint32_t ranges = 1;
  if (n > kRankMost)
    while (ranges < kMostRanges && (uint64_t)ranges * kRangeKeys < n) ranges <<= 1;
  const uint32_t ranked = ranges > 1 ? ranges * kOversample : (uint32_t)n;
  uint64_t* bounds = ranges > 1 ? ws.key[1] : nullptr;
  const uint32_t per_block = kThreads / kRankLanes;
  hipLaunchKernelGGL(export_rank_kernel, dim3((ranked + per_block - 1) / per_block), dim3(kThreads), 0, stream, ws,
                     (uint32_t)n / ranked, ranked, out, bounds);
  if (ranges > 1)
    hipLaunchKernelGGL(export_ranges_kernel, dim3(ranges), dim3(kRangeThreads), 0, stream, ws, (uint32_t)n, ranges, bounds, out);
  return hipGetLastError();
}

}  // namespace mono
