// lookup_or_insert for small batches (at most kSmallLookup keys): one launch.
//
// The general path is three kernels (four for large batches), because counting, election and placement each need the one
// before finished on the whole chip.  A batch of a few thousand keys is nothing but their latency: 1700 keys
// that the table knows took 5.4 + 1.8 + 2.1 + 2.8 us in four kernels and about as much again between them.
// Here every block probes 128 keys with 512 threads (eight lanes per key, both of its buckets requested at
// once: a small batch has no bandwidth to save), stamps the hits, counts the misses, and hands the missing
// occurrences to the block that finishes last, which elects, places and resolves them alone, with the set of
// distinct missing keys in LDS.  A batch without misses, the usual one when serving, ends with the probe.
// (Known keys, GPU time of a call of 200, 1088 and 4096 with 256 keys and 1024 threads: 4.7, 5.2, 5.3 us; with 128 and 512:
// 4.3, 4.6, 4.7; with 64 and 256: 4.5, 4.6, 5.0.)
// 4096 keys that the table knows, or nearly all, take half the time of 5000 in three kernels (dim 32: 5 to 7 and 14 to 16 us;
// with 1 % unknown 10 to 14 and 16 to 22, 5 % 12 to 16 and 18 to 24); from a third of them unknown on one block's work costs as
// much as the launches it saves (30 % 16 to 30 and 21 to 26), and all of them, where they are admitted, twice as much (54 to 68
// and 31; 27 and 24 where they are not).
// (Lookups with 5, 30 and 100 % new keys, dim 16, 2^22 slots, us, with the eight exchanges of an insertion unrolled and every
// bucket's age byte read, and as they are now, see try_claim: 200 IDs 12.4 / 11.0, 14.4 / 11.9, 15.7 / 13.2, 1000 14.0 / 11.6,
// 15.6 / 12.9, 24.2 / 19.9, 4096 16.4 / 13.7, 29.3 / 22.9, 73 / 54; with expiry 13.8 / 12.1 to 17.3 / 14.5, 15.6 / 12.8 to
// 27.3 / 21.5, 17.9 / 14.9 to 85 / 58.)
//
// Blocks run on different XCDs, whose L2s are not coherent for ordinary accesses.  What a block leaves for
// the last one in this same kernel (missing occurrences, counters, last-seen stamps that an eviction may
// move) goes through agent-scope atomics, and a block reports itself done only after its waves have waited
// for theirs.  Only the first values of new rows are not left to that block: they are hashes, 20 us of one block for a
// thousand rows of dim 128.  Blocks that know of a miss when they finish stay, look for the list of new rows and share it
// (1088 IDs of dim 128, half of them new: 70 -> 60 us for a training step; lookups with that block alone and so, 200 and 4096
// IDs of which 5 % are new, dim 16 10.5 / 10.6 and 14.4 / 14.4 us, dim 32 11.6 / 12.0 and 16.3 / 14.8, dim 128 14.0 / 12.1 and
// 23.7 / 15.3; 30 % new, dim 16 12.4 / 11.7 and 24.3 / 24.1, dim 128 21.5 / 14.2 and 49 / 25).  They wait a bounded time, and
// nothing depends on them: every block has counted itself done before it waits, and a list that nobody helps with the last block does.
#include "common.h"
#include "kernels.h"
#include "table_ops.h"

namespace mono {

constexpr int kSmallThreads = 512, kSmallKeysPerBlock = 128;
constexpr uint32_t kSmallChunk = 16;   // new rows that a wave initialises at a time
constexpr int kSmallPolls = 4096;      // looks of a waiting block at the last block's word: some milliseconds
constexpr uint32_t kSmallSet = 2 * kSmallKeysPerBlock;  // slots of a block's set of missing keys
static_assert(kSmallThreads == 4 * kSmallKeysPerBlock, "two keys per group of eight lanes");
constexpr int kSmallPerThread = (int)(kSmallLookup / kSmallThreads);

struct SmallProbe {
  unsigned long long miss_key[kSmallSet];
  uint32_t miss_cnt[kSmallSet];
  unsigned long long key[kSmallKeysPerBlock];  // missing occurrences of this block
  uint32_t occ[kSmallKeysPerBlock];
};
struct SmallFinish {
  unsigned long long key[kSmallLookup];  // the batch's missing occurrences
  alignas(16) uint32_t slot[4 * kSmallLookup];  // set of distinct missing keys (number of the first occurrence); later: the winners
  int32_t row[kSmallLookup];             // what a leader found for its key
};

// Initialises new rows from the list that the last block has left, in chunks that the waves of all blocks take in turn.
template <typename E>
__device__ inline void init_listed_rows(const TableView& t, uint32_t total) {
  const uint32_t lane = lane_id();
  const RestoreSource none = {nullptr, nullptr, nullptr};
  for (;;) {  // (every turn takes a chunk: at most total / kSmallChunk turns and one)
    unsigned long long chunk = 0;
    if (lane == 0) chunk = atomicAdd(&t.ctl->scratch[kSmallNext], 1ull);
    const uint32_t w0 = (uint32_t)__shfl(chunk, 0) * kSmallChunk;
    if (w0 >= total) return;
    const bool mine = lane < kSmallChunk && w0 + lane < total;
    uint64_t key = kEmptyKey;
    uint32_t row = kNoRow;
    if (mine) {
      const unsigned long long* from = reinterpret_cast<const unsigned long long*>(&t.win_list[w0 + lane]);
      key = ld_agent(from);
      row = (uint32_t)ld_agent(from + 1);
    }
    init_new_rows<E>(t, mine, kSmallChunk, key, row, 0u, none);
  }
}

template <typename E>
__global__ __launch_bounds__(kSmallThreads) void lookup_small_kernel(TableView t, const int64_t* __restrict__ keys,
                                                                     uint32_t n, uint32_t step, uint32_t epoch,
                                                                     int32_t* __restrict__ rows_out) {
  __shared__ union {
    SmallProbe p;
    SmallFinish f;
  } s;
  __shared__ uint32_t s_count, s_base, s_last;
  __shared__ uint32_t s_wave[kSmallThreads / 64];
  const uint32_t tid = threadIdx.x, lane = lane_id(), gi = lane & 7u, gbase = lane & ~7u;
  if (tid < kSmallSet) {
    s.p.miss_key[tid] = kEmptyKey;
    s.p.miss_cnt[tid] = 0;
  }
  if (tid == 0) s_count = 0;
  // ---- probe: group of eight lanes <-> two keys, four bucket lines in flight ------------------------
  constexpr int kTurns = 2;
  uint32_t occ[kTurns];
  uint64_t k[kTurns], b0[kTurns], b1[kTurns];
  ulonglong2 d0[kTurns], d1[kTurns];
#pragma unroll
  for (int r = 0; r < kTurns; ++r) {
    occ[r] = blockIdx.x * kSmallKeysPerBlock + (uint32_t)r * (kSmallThreads / 8) + (tid >> 3);
    k[r] = occ[r] < n ? (uint64_t)keys[occ[r]] : kEmptyKey;
  }
#pragma unroll
  for (int r = 0; r < kTurns; ++r) {
    b0[r] = bucket_index(t, 0, k[r]);
    b1[r] = bucket_index(t, 1, k[r]);
    d0[r] = reinterpret_cast<const ulonglong2*>(t.buckets + b0[r])[gi];
    d1[r] = reinterpret_cast<const ulonglong2*>(t.buckets + b1[r])[gi];
  }
  const uint32_t sn = t.ctl->stash_n;
  __syncthreads();  // the set is cleared
#pragma unroll
  for (int r = 0; r < kTurns; ++r) {
    const bool live = k[r] != kEmptyKey, key_lane = live && gi < 4;
    // lanes 0-3 of the group hold the bucket's keys two by two, lanes 4-7 the meta words
    const uint32_t x0 = (uint32_t)(__ballot(key_lane && d0[r].x == k[r]) >> gbase) & 0xFu;
    const uint32_t y0 = (uint32_t)(__ballot(key_lane && d0[r].y == k[r]) >> gbase) & 0xFu;
    const uint32_t x1 = (uint32_t)(__ballot(key_lane && d1[r].x == k[r]) >> gbase) & 0xFu;
    const uint32_t y1 = (uint32_t)(__ballot(key_lane && d1[r].y == k[r]) >> gbase) & 0xFu;
    const bool in0 = (x0 | y0) != 0, hit = in0 || (x1 | y1) != 0;
    const uint32_t x = in0 ? x0 : x1, y = in0 ? y0 : y1;
    const int pair = hit ? __ffs((int)(x | y)) - 1 : 0;
    const int slot = 2 * pair + (x ? 0 : 1);
    const unsigned long long mx = in0 ? d0[r].x : d1[r].x, my = in0 ? d0[r].y : d1[r].y;
    const unsigned long long m = x ? __shfl(mx, (int)gbase + 4 + pair) : __shfl(my, (int)gbase + 4 + pair);
    if (gi != 0 || occ[r] >= n) continue;
    if (!live) {
      rows_out[occ[r]] = kRowAbsent;
    } else if (hit) {
      rows_out[occ[r]] = (int32_t)meta_row(m);
      if (meta_seen(m) != step)
        st_agent(reinterpret_cast<uint32_t*>(&t.buckets[in0 ? b0[r] : b1[r]].meta[slot]) + 1, step);  // stamp
    } else {
      bool miss = true;
      const uint32_t lim = sn < kStashCap ? sn : kStashCap;
      for (uint32_t q = 0; q < lim && miss; ++q)
        if (t.stash[q].key == k[r]) {
          rows_out[occ[r]] = (int32_t)t.stash[q].row;
          t.stash[q].seen = step;
          miss = false;
        }
      if (miss) {
        uint32_t pos = (uint32_t)(mix64(k[r] ^ t.s_dedup) >> 40) & (kSmallSet - 1);
        for (;;) {  // at most half of the slots are ever taken: a free slot always turns up
          const unsigned long long old = atomicCAS(&s.p.miss_key[pos], (unsigned long long)kEmptyKey, (unsigned long long)k[r]);
          if (old == kEmptyKey || old == k[r]) break;
          pos = (pos + 1) & (kSmallSet - 1);
        }
        atomicAdd(&s.p.miss_cnt[pos], 1u);
        const uint32_t at = atomicAdd(&s_count, 1u);
        s.p.key[at] = k[r];
        s.p.occ[at] = occ[r];
      }
    }
  }
  __syncthreads();
  const uint32_t mine = s_count;
  if (mine) {  // block-uniform
    if (tid == 0) s_base = (uint32_t)atomicAdd(&t.ctl->scratch[kSmallMisses], (unsigned long long)mine);
    if (tid < kSmallSet && s.p.miss_cnt[tid]) touch_counter<false>(t, s.p.miss_key[tid], step, s.p.miss_cnt[tid]);
    __syncthreads();
    if (tid < mine) {
      unsigned long long* to = reinterpret_cast<unsigned long long*>(&t.win_list[s_base + tid]);
      st_agent(to, s.p.key[tid]);
      st_agent(to + 1, (unsigned long long)s.p.occ[tid]);
    }
  }
  wait_all_memory_ops();  // stamps, counters and list entries of this wave are performed
  __syncthreads();
  if (tid == 0) {  // low half: blocks done; high half: their missing occurrences
    const unsigned long long before = atomicAdd(&t.ctl->scratch[kSmallDone], (unsigned long long)mine << 32 | 1ull);
    s_last = (uint32_t)before == gridDim.x - 1;
    s_count = 0;
    if (!s_last && ((before >> 32) != 0 || mine)) {
      // Someone misses: stay for the list of new rows that the last block makes of it, but not for ever.
      for (int poll = 0; poll < kSmallPolls; ++poll) {
        const unsigned long long go = ld_agent(&t.ctl->scratch[kSmallGo]);
        if ((uint32_t)(go >> 32) == epoch) {
          s_count = (uint32_t)go;
          break;
        }
        __builtin_amdgcn_s_sleep(8);
      }
    }
  }
  __syncthreads();
  if (!s_last) {
    if (s_count) init_listed_rows<E>(t, s_count);
    return;
  }

  // ---- the block that finished last: everything about the missing occurrences -----------------------
  if (tid == 0) {
    s_count = (uint32_t)ld_agent(&t.ctl->scratch[kSmallMisses]);
    t.ctl->scratch[kSmallMisses] = 0;  // for the next call
    t.ctl->scratch[kSmallDone] = 0;
  }
  __syncthreads();
  const uint32_t missed = s_count;
  if (missed == 0) {
    // (the mark has not moved; the host only wants to hear of a call now and then, and the store over the bus holds
    // the kernel's end: 7.5 -> 6.9 us for 1700 known keys)
    if (tid == 0 && t.hwm_mail && epoch % kPostEvery == 0) post_hwm(t, epoch, t.ctl->hwm);
    return;
  }
  // Four slots for each: the slowest of a wave's 64 keys then finds its place in three or four steps, with two slots for each in
  // seven or eight, and a thread has up to eight keys (4096 unknown keys below the threshold 32 -> 27 us, admitted 59 -> 54).
  uint32_t slots = 64;
  while (slots < 4 * missed) slots <<= 1;
  for (uint32_t q = 4 * tid; q < slots; q += 4 * kSmallThreads)
    *reinterpret_cast<uint4*>(&s.f.slot[q]) = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  uint64_t mk[kSmallPerThread];
  uint32_t mo[kSmallPerThread], lead[kSmallPerThread];
#pragma unroll
  for (int j = 0; j < kSmallPerThread; ++j) {
    const uint32_t x = (uint32_t)j * kSmallThreads + tid;
    mk[j] = kEmptyKey;
    if (x < missed) {
      const unsigned long long* from = reinterpret_cast<const unsigned long long*>(&t.win_list[x]);
      mk[j] = ld_agent(from);
      mo[j] = (uint32_t)ld_agent(from + 1);
      s.f.key[x] = mk[j];
    }
  }
  wait_all_memory_ops();  // (the list is written over below, and nothing else waits for the last occurrence number)
  __syncthreads();
  uint32_t cnt[kSmallPerThread];
#pragma unroll
  for (int j = 0; j < kSmallPerThread; ++j) {
    const uint32_t x = (uint32_t)j * kSmallThreads + tid;
    lead[j] = x;
    cnt[j] = 0;
    if (x >= missed) continue;
    uint32_t pos = (uint32_t)(mix64(mk[j] ^ t.s_dedup) >> 32) & (slots - 1);
    for (;;) {  // at most a quarter of the slots is ever taken: a free slot always turns up
      const uint32_t old = atomicCAS(&s.f.slot[pos], 0xFFFFFFFFu, x);
      if (old == 0xFFFFFFFFu) break;
      if (s.f.key[old] == mk[j]) {
        lead[j] = old;
        break;
      }
      pos = (pos + 1) & (slots - 1);
    }
    if (lead[j] != x) continue;
    cnt[j] = 255u;  // (with a threshold of 0 or 1 every missing key is admissible)
    if (t.freq_threshold > 1u)
      for (uint32_t h = 0; h < t.filter_hashes; ++h) {  // smallest of the key's counters, read as min(count, 255)
        const uint32_t c = ld_agent(reinterpret_cast<const uint32_t*>(&t.filter[filter_index(t, mk[j], h)]));
        cnt[j] = c < cnt[j] ? c : cnt[j];
      }
  }
  // rank of every winner among the winners of the call
  uint32_t below = 0, of_wave = 0;
  uint32_t rank[kSmallPerThread];
  bool wins[kSmallPerThread];
#pragma unroll
  for (int j = 0; j < kSmallPerThread; ++j) {
    const uint32_t x = (uint32_t)j * kSmallThreads + tid;
    wins[j] = x < missed && lead[j] == x && cnt[j] >= t.freq_threshold;
    const uint64_t m = __ballot(wins[j]);
    rank[j] = of_wave + (uint32_t)__popcll(m & lanes_below());
    of_wave += (uint32_t)__popcll(m);
  }
  if (lane == 0) s_wave[tid >> 6] = of_wave;
  __syncthreads();  // (and nobody needs the set any more)
  uint32_t total = 0;
  for (uint32_t w = 0; w < kSmallThreads / 64; ++w) {
    if (w == (tid >> 6)) below = total;
    total += s_wave[w];
  }
  const int32_t free0 = t.ctl->free_n;
  const uint32_t hwm0 = t.ctl->hwm;
  // all of the call's new keys fit under the fill limit, or none of them is placed
  const bool room = (int64_t)total <= rows_on_offer(t.capacity, free0);
#pragma unroll
  for (int j = 0; j < kSmallPerThread; ++j) {
    const uint32_t x = (uint32_t)j * kSmallThreads + tid;
    if (x >= missed || lead[j] != x) continue;
    int32_t row = kRowAbsent;
    if (wins[j]) {
      if (room) row = (int32_t)t.free_rows[free0 - 1 - (int32_t)(below + rank[j])];
      s.f.slot[below + rank[j]] = x;
    }
    s.f.row[x] = row;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallPerThread; ++j) {
    const uint32_t x = (uint32_t)j * kSmallThreads + tid;
    if (x < missed) rows_out[mo[j]] = s.f.row[lead[j]];
  }
  // The list of new rows goes to the blocks that wait for it, and this one joins them when it has placed the keys.
  const uint32_t placed = room ? total : 0u;
  for (uint32_t w = tid; w < placed; w += kSmallThreads) {
    const uint32_t x = s.f.slot[w];
    unsigned long long* to = reinterpret_cast<unsigned long long*>(&t.win_list[w]);
    st_agent(to, s.f.key[x]);
    st_agent(to + 1, (unsigned long long)(uint32_t)s.f.row[x]);
  }
  if (tid == 0) st_agent(&t.ctl->scratch[kSmallNext], 0ull);
  wait_all_memory_ops();
  __syncthreads();
  if (tid == 0) st_agent(&t.ctl->scratch[kSmallGo], (unsigned long long)epoch << 32 | placed);
  for (uint32_t w = tid; w < placed; w += kSmallThreads) {
    const uint32_t x = s.f.slot[w];
    cuckoo_insert(t, s.f.key[x], make_meta((uint32_t)s.f.row[x], step), sweep_unit(step, t.sweep_q));
  }
  if (placed) init_listed_rows<E>(t, placed);
  if (tid == 0) settle_call(t, total, free0, hwm0, epoch);
}

hipError_t launch_lookup_small(const TableView& t, const int64_t* d_keys, uint64_t n, uint32_t step, uint32_t epoch,
                               int32_t* d_rows_out, hipStream_t stream, Profiler* prof) {
  const dim3 grid((unsigned)((n + kSmallKeysPerBlock - 1) / kSmallKeysPerBlock)), block(kSmallThreads);
  if (t.bf16)
    MONO_LAUNCH(prof, K_LOOKUP_SMALL, stream, lookup_small_kernel<uint16_t>, grid, block, t, d_keys, (uint32_t)n, step, epoch,
                d_rows_out);
  else
    MONO_LAUNCH(prof, K_LOOKUP_SMALL, stream, lookup_small_kernel<float>, grid, block, t, d_keys, (uint32_t)n, step, epoch,
                d_rows_out);
  return hipGetLastError();
}

}  // namespace mono
