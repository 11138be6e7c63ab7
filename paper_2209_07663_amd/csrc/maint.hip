// Expiry sweep (paper section 2.1, second heuristic: IDs inactive for a configured time are
// removed), plus the untimed maintenance kernels: initialisation, table dump (all keys, or only the
// keys trained in the current synchronisation window: section 2.2.3), counter dump and counter restore.
#include "common.h"
#include "kernels.h"

namespace mono {

__device__ inline bool is_expired(const TableView& t, uint32_t now, uint32_t seen) {
  return t.expire_steps > 0 && now >= seen && now - seen >= t.expire_steps;
}

// Sweep in two kernels, or where the table is small and nobody asks for the keys in one that does both (sweep_small):
//   sweep_find    reads the bound of every bucket (a byte each, kept by insertions and by the sweep itself) and looks
//                 only at buckets that may hold a key that is too old; takes such keys out of their slots,
//                 appends their rows to one of kWinLists lists (one atomic per wave and 64 buckets, spread
//                 over the lists) and writes the bucket's new bound.  A key that nobody sees again is looked
//                 at once, when it expires; a bucket of keys that stay in use about once in expire_steps.
//                 (Before there were bounds a sweep read every bucket that was not empty: 129 us of a
//                 2^25-slot table at load 0.7, 81 us of 2^28 slots with 3.6 M keys.)  One thread also walks the
//                 (normally empty) stash.
//   sweep_remove  dense over the lists: pushes the rows on the free stack by rank; the block that finishes last settles
//                 the counters.  Where the caller wants the removed keys, the lists hold slots and this
//                 kernel reports the keys and clears the slots.
__device__ inline void sweep_stash(const TableView& t, uint32_t now, int64_t* expired_keys, uint64_t max_expired) {
  Control* c = t.ctl;
  unsigned long long removed = 0;
  uint32_t sn = c->stash_n < kStashCap ? c->stash_n : kStashCap;
  if (c->stash_n) {
    for (uint32_t s = 0; s < sn;) {
      if (is_expired(t, now, t.stash[s].seen)) {
        if (expired_keys && removed < max_expired) expired_keys[removed] = (int64_t)t.stash[s].key;
        t.free_rows[c->free_n] = t.stash[s].row;
        c->free_n += 1;
        t.stash[s] = t.stash[sn - 1];
        --sn;
        ++removed;
      } else {
        ++s;
      }
    }
    c->stash_n = sn;
  }
  c->scratch[kSweepRemoved] = removed;
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Which bounds (bytes of `oldest`) mean that a bucket may hold a key that is too old: a byte in [0, low) or in
// [from, from + many).  Bounds go round, so that the young ones, from now's back to the oldest that is still young, are one
// interval or the two ends of 1..254; 0 (kAgeLook) is looked at and 255 (kAgeEmpty) never.  Two bytes an instruction: with
// the age of every byte worked out alone, 2^28 slots were bound by instructions (32 waves of 400 each to a SIMD, 20 us).
struct OldBounds {
  uint32_t low, from, many;
  __device__ OldBounds(const TableView& t, uint32_t now, bool all) {
    const uint32_t unit_now = now >> t.sweep_q, rest = now - (unit_now << t.sweep_q), here = sweep_unit(now, t.sweep_q);
    // the greatest age in units of which even the first step is less than expire_steps ago
    const uint32_t units = min((t.expire_steps - 1u - rest) >> t.sweep_q, unit_now);
    low = all ? 255u : (here > units ? here - units : 1u);
    from = here + 1u;
    many = all ? 0u : (here > units ? 254u - here : 253u - units);
  }
  // two bytes in the halves of x: 1 in the halves of those
  __device__ uint32_t operator()(uint32_t x) const {
    const u16x2 v = __builtin_bit_cast(u16x2, x), one = (uint16_t)1;
    const u16x2 found = __builtin_elementwise_sub_sat((u16x2)(uint16_t)low, v) |
                        __builtin_elementwise_sub_sat((u16x2)(uint16_t)many, (u16x2)(v - (u16x2)(uint16_t)from));
    return __builtin_bit_cast(uint32_t, (u16x2)__builtin_elementwise_min(found, one));
  }
};

// smallest value of the group of eight lanes (called by whole waves)
__device__ inline uint32_t least_of_eight(uint32_t x) {
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false));   // lane ^ 1
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false));   // lane ^ 2
  return min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false));  // 7 - lane
}

constexpr int kSweepTurns = 8;  // buckets per group of eight lanes with their meta words (64 bytes) in flight

// The wave's list of buckets to look at, from the bounds of kWords * 256 of them, and how many they are.
template <int kWords>
__device__ inline uint32_t list_old_buckets(const uint32_t (&word)[kWords], const OldBounds& is_old, uint16_t* list) {
  uint32_t look = 0;  // one bit per bucket of the lane's; bit 16 h + 2 w + o: byte 2 h + o of word w
#pragma unroll
  for (int w = 0; w < kWords; ++w)
    look |= is_old(word[w] & 0x00FF00FFu) << (2 * w) | is_old((word[w] >> 8) & 0x00FF00FFu) << (2 * w + 1);
  if (__ballot(look != 0) == 0) return 0;  // wave-uniform
  const uint32_t inc = wave_sums((uint32_t)__popc(look));
  wave_order();
  uint32_t at = inc - (uint32_t)__popc(look);
  for (uint32_t m = look; m; m &= m - 1) {
    const uint32_t i = (uint32_t)__ffs((int)m) - 1u;
    wave_store(list + at++, (uint16_t)(lane_id() * (4 * kWords) + ((i >> 1) & 7u) * 4u + (i >> 4) * 2u + (i & 1u)));
  }
  wave_order();
  return lane_value(inc, 63);
}

// Looks at 8 * kSweepTurns buckets of the list, from e0 on, and writes their new bounds.  m: meta words; gone: the lanes whose
// keys are too old; returns how many.
__device__ inline uint32_t look_at_buckets(const TableView& t, uint32_t now, uint64_t bucket0, const uint16_t* list, uint32_t e0,
                                           uint32_t total, unsigned long long (&m)[kSweepTurns], uint64_t (&gone)[kSweepTurns]) {
  const uint32_t grp = lane_id() >> 3, l8 = lane_id() & 7;
#pragma unroll
  for (int r = 0; r < kSweepTurns; ++r) {
    const uint32_t e = e0 + 8u * (uint32_t)r + grp;
    m[r] = kNoMeta;
    if (e < total) m[r] = t.buckets[bucket0 + wave_load(list + e)].meta[l8];
  }
  uint32_t found = 0;
#pragma unroll
  for (int r = 0; r < kSweepTurns; ++r) {
    gone[r] = 0;
    if (e0 + 8u * (uint32_t)r >= total) continue;  // wave-uniform
    const uint32_t e = e0 + 8u * (uint32_t)r + grp;
    const bool live = meta_row(m[r]) != kNoRow, old = live && is_expired(t, now, meta_seen(m[r]));
    gone[r] = __ballot(old);
    found += (uint32_t)__popcll(gone[r]);
    const uint32_t least = least_of_eight(live && !old ? meta_seen(m[r]) : 0xFFFFFFFFu);  // over the keys that stay
    if (e < total && l8 == 0) {
      const uint64_t b = bucket0 + wave_load(list + e);
      // (a key from the future, seen after `now`: nothing is known)
      const uint32_t age = least == 0xFFFFFFFFu ? kAgeEmpty : (least > now ? kAgeLook : sweep_unit(least, t.sweep_q));
      reinterpret_cast<uint8_t*>(t.oldest)[b] = (uint8_t)age;
      if (age == kAgeEmpty) atomicAnd(&t.occupied[b >> 6], ~(1ull << (b & 63)));
    }
  }
  return found;
}

// Hands out the keys that are gone: calls `each` with their numbers from p on, buckets, slots and meta words.
template <typename F>
__device__ inline void each_gone(uint64_t bucket0, const uint16_t* list, uint32_t e0, const unsigned long long (&m)[kSweepTurns],
                                 const uint64_t (&gone)[kSweepTurns], uint32_t p, const F& each) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int r = 0; r < kSweepTurns; ++r) {
    if (gone[r] == 0) continue;  // wave-uniform
    if ((gone[r] >> lane) & 1ull)
      each(p + (uint32_t)__popcll(gone[r] & lanes_below()), bucket0 + wave_load(list + e0 + 8u * (uint32_t)r + (lane >> 3)), m[r]);
    p += (uint32_t)__popcll(gone[r]);
  }
}

// Bounds are unambiguous while every key's last-seen step lies in the last kAgeModulus units: all keys that the
// latest sweep left were seen less than expire_steps before it.  Beyond that every bucket is looked at, as it is
// where the caller's steps went back behind the latest sweep (`now` did, or a lookup in between: look_all).
__device__ inline bool looks_at_all(const TableView& t, uint32_t now, bool look_all) {
  const uint32_t unit_now = now >> t.sweep_q, swept = t.ctl->swept;
  const uint32_t unit_least = (swept > t.expire_steps ? swept - t.expire_steps : 0u) >> t.sweep_q;
  return look_all || unit_now - unit_least >= kAgeModulus - 1 || now < swept;
}

// The bounds of the lane's buckets of a share of 256 * kWords; kAgeEmpty beyond the table's n.
template <int kWords>
__device__ inline void load_bounds(const TableView& t, uint64_t share, uint64_t n, uint32_t (&word)[kWords]) {
#pragma unroll
  for (int w = 0; w < kWords; ++w) word[w] = 0xFFFFFFFFu;
  const uint64_t first = share * (256u * kWords) + (uint64_t)lane_id() * (4 * kWords);  // the lane's buckets
  if (first + 4 * kWords <= n) {
    if constexpr (kWords == 4) {
      const uint4 q = *reinterpret_cast<const uint4*>(t.oldest + (first >> 2));
      word[0] = q.x;
      word[1] = q.y;
      word[2] = q.z;
      word[3] = q.w;
    } else {
      word[0] = t.oldest[first >> 2];
    }
  } else {
    for (uint32_t j = 0; j < 4 * kWords && first + j < n; ++j) {  // (tables of fewer than 2048 slots)
      const uint32_t byte = reinterpret_cast<const uint8_t*>(t.oldest)[first + j];
      word[j >> 2] = (word[j >> 2] & ~(0xFFu << (8 * (j & 3)))) | (byte << (8 * (j & 3)));
    }
  }
}

// kWords: words of four bounds per lane, so that a wave takes 256 * kWords buckets at a time.  Four of them (16-byte loads)
// on large tables, whose bounds are then a plain stream; one on small tables, which would have too few waves.
// keep_slots: the lists take slots and the slots stay as they are (see sweep_remove).
template <int kWords>
__global__ __launch_bounds__(256) void sweep_find_kernel(TableView t, uint32_t now, bool look_all, int keep_slots,
                                                         int64_t* expired_keys, uint64_t max_expired) {
  constexpr uint32_t kBuckets = 256u * kWords;
  __shared__ uint16_t s_list[4][kBuckets];
  if (blockIdx.x == 0 && threadIdx.x == 0) sweep_stash(t, now, expired_keys, max_expired);
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  const uint64_t n = 2 * t.n_buckets;
  const uint32_t shares = (uint32_t)((n + kBuckets - 1) / kBuckets), step = gridDim.x * 4;
  uint32_t share = blockIdx.x * 4 + wave;
  if (share >= shares) return;  // wave-uniform (no barriers below)
  uint32_t word[kWords];
  load_bounds<kWords>(t, share, n, word);
  const OldBounds is_old(t, now, looks_at_all(t, now, look_all));
  uint16_t* list = s_list[wave];  // the buckets to look at, of the wave's
  while (share < shares) {
    const uint64_t bucket0 = (uint64_t)share * kBuckets;
    const uint32_t out = share & (kWinLists - 1);  // the sub-list
    const uint32_t total = list_old_buckets<kWords>(word, is_old, list);
    share += step;
    load_bounds<kWords>(t, share, n, word);  // (nothing beyond the last share)
    for (uint32_t e0 = 0; e0 < total; e0 += 8 * kSweepTurns) {
      unsigned long long m[kSweepTurns];
      uint64_t gone[kSweepTurns];
      const uint32_t found = look_at_buckets(t, now, bucket0, list, e0, total, m, gone);
      if (found == 0) continue;  // wave-uniform
      uint32_t p = 0;
      if (lane == 0) p = atomicAdd(&t.sweep_cnt[out * kWinStride], found);
      p = __shfl(p, 0);
      each_gone(bucket0, list, e0, m, gone, p, [&](uint32_t at, uint64_t b, unsigned long long meta) {
        const uint32_t l8 = lane_id() & 7;
        t.sweep_list[(uint64_t)out * t.sweep_cap + at] = keep_slots ? (uint32_t)(b * kBucket + l8) : meta_row(meta);
        if (!keep_slots) {
          t.buckets[b].meta[l8] = kNoMeta;
          t.buckets[b].key[l8] = kEmptyKey;
        }
      });
    }
  }
}

// Both in one, for tables of few blocks whose caller does not ask for the removed keys: a block adds what it has found to one
// word, at most four times, which gives it its place on the free stack; the block that comes last settles the counters.
// One word takes an addition every 12 ns, so that with more blocks they wait for it as long as a launch takes (both kernels and
// this one: 2^13 slots 11.9 and 8.7 us, 2^22 slots 9.4 and 5.8; training steps of 2^20 slots 64.6 and 60.8, 2^23 slots 112 and
// 108; with 512 blocks for 2^24 slots 248.6 and 249.6, with 1024 for 2^25, a million keys removed, 1122 and 1128).
constexpr int kSweepSmallThreads = 1024, kSweepSmallWaves = kSweepSmallThreads / 64;
constexpr uint64_t kSweepSmallBlocks = 256;  // 2^23 slots

__global__ __launch_bounds__(kSweepSmallThreads) void sweep_small_kernel(TableView t, uint32_t now, bool look_all,
                                                                         uint64_t* n_expired) {
  __shared__ uint16_t s_list[kSweepSmallWaves][256];
  __shared__ uint32_t s_found[kSweepSmallWaves], s_rounds;
  __shared__ unsigned long long s_before;
  const uint32_t wave = threadIdx.x >> 6, share = blockIdx.x * kSweepSmallWaves + wave;
  uint32_t word[1];
  load_bounds<1>(t, share, 2 * t.n_buckets, word);
  // settled by the last block, constant until then
  const int32_t free0 = t.ctl->free_n;
  const uint32_t in_stash = t.ctl->stash_n;
  const unsigned long long expired0 = t.ctl->n_expired;
  const OldBounds is_old(t, now, looks_at_all(t, now, look_all));
  if (threadIdx.x == 0) s_rounds = 1;
  __syncthreads();
  uint16_t* list = s_list[wave];
  const uint64_t bucket0 = (uint64_t)share * 256u;
  const uint32_t total = list_old_buckets<1>(word, is_old, list);
  if (total > 8 * kSweepTurns && lane_id() == 0) atomicMax(&s_rounds, (total + 8 * kSweepTurns - 1) / (8 * kSweepTurns));
  __syncthreads();
  const uint32_t rounds = s_rounds;
  unsigned long long removed = 0;  // by this block and those before it
  for (uint32_t round = 0; round < rounds; ++round) {  // block-uniform
    const uint32_t e0 = round * 8 * kSweepTurns;
    unsigned long long m[kSweepTurns];
    uint64_t gone[kSweepTurns];
    uint32_t found = 0;
    if (e0 < total) found = look_at_buckets(t, now, bucket0, list, e0, total, m, gone);  // wave-uniform
    if (lane_id() == 0) s_found[wave] = found;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (uint32_t w = 0; w < (uint32_t)kSweepSmallWaves; ++w) {
      if (w == wave) before = all;
      all += s_found[w];
    }
    // high half: keys removed; low half: blocks done
    if (threadIdx.x == 0)
      s_before = atomicAdd(&t.ctl->scratch[kSweepDone], (unsigned long long)all << 32 | (round == rounds - 1 ? 1ull : 0ull));
    __syncthreads();
    const uint32_t first = (uint32_t)(s_before >> 32);
    removed = (unsigned long long)first + all;
    if (found)
      each_gone(bucket0, list, e0, m, gone, first + before, [&](uint32_t at, uint64_t b, unsigned long long meta) {
        t.free_rows[free0 + (int32_t)at] = meta_row(meta);
        t.buckets[b].meta[lane_id() & 7] = kNoMeta;
        t.buckets[b].key[lane_id() & 7] = kEmptyKey;
      });
  }
  if (threadIdx.x != 0 || (uint32_t)s_before != gridDim.x - 1) return;
  t.ctl->scratch[kSweepDone] = 0;
  t.ctl->free_n = free0 + (int32_t)removed;
  t.ctl->swept = now;
  if (in_stash) {
    sweep_stash(t, now, nullptr, 0);  // (counts on from there)
    removed += t.ctl->scratch[kSweepRemoved];
  }
  t.ctl->n_expired = expired0 + removed;
  if (n_expired) *n_expired = removed;
}

// expired_keys != nullptr: the lists hold slots, which are cleared here.
__global__ __launch_bounds__(256) void sweep_remove_kernel(TableView t, uint32_t now, int64_t* expired_keys,
                                                           uint64_t max_expired, uint64_t* n_expired) {
  const uint32_t lane = lane_id();
  const uint32_t inc = wave_sums(t.sweep_cnt[lane * kWinStride]);
  const uint32_t total = lane_value(inc, 63);
  const int32_t free0 = t.ctl->free_n;                     // settled by the last block, constant until then
  const unsigned long long out0 = t.ctl->scratch[kSweepRemoved];       // keys already reported from the stash
  const uint32_t stride = gridDim.x * blockDim.x;
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * blockDim.x + (threadIdx.x & ~63u)));
  for (uint32_t w0 = first; w0 < total; w0 += stride) {
    const uint32_t w = w0 + lane;
    uint32_t before;
    const uint32_t list = list_holding(inc, w, w0, w < total, &before);
    if (w < total) {
      uint32_t g = t.sweep_list[(uint64_t)list * t.sweep_cap + (w - before)];
      if (expired_keys) {
        Bucket* b = &t.buckets[g >> 3];
        const int l = (int)(g & 7);
        g = meta_row(b->meta[l]);
        if (out0 + w < max_expired) expired_keys[out0 + w] = (int64_t)b->key[l];
        b->meta[l] = kNoMeta;
        b->key[l] = kEmptyKey;
      }
      t.free_rows[free0 + (int32_t)w] = g;
    }
  }
  // The block that finishes last settles the counters: the others have read them.  (Blocks count themselves on the
  // counters' 64 lines first, and the last of each line on one word: one word alone would serialise thousands
  // of them at ~12 ns each.)
  __syncthreads();
  if (threadIdx.x != 0) return;
  const uint32_t line = blockIdx.x & (kWinLists - 1);
  const uint32_t of_line = (gridDim.x - line + kWinLists - 1) / kWinLists, lines = gridDim.x < kWinLists ? gridDim.x : kWinLists;
  if (atomicAdd(&t.sweep_cnt[line * kWinStride + 1], 1u) != of_line - 1) return;
  if (atomicAdd(&t.ctl->scratch[kSweepDone], 1ull) != (unsigned long long)lines - 1) return;
  for (int l = 0; l < kWinLists; ++l) *reinterpret_cast<uint2*>(&t.sweep_cnt[l * kWinStride]) = make_uint2(0u, 0u);
  t.ctl->scratch[kSweepDone] = 0;
  t.ctl->free_n = free0 + (int32_t)total;
  t.ctl->swept = now;
  const unsigned long long removed = out0 + total;
  t.ctl->n_expired += removed;
  if (n_expired) *n_expired = removed;
}

__global__ void sweep_nothing_kernel(uint64_t* n_expired) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *n_expired = 0;
}

constexpr uint64_t kSweepBlocks = 4096;

hipError_t launch_expire_sweep(const TableView& t, uint32_t now, bool look_all, uint64_t* d_n_expired,
                               int64_t* d_expired_keys, uint64_t max_expired, hipStream_t stream, Profiler* prof) {
  if (t.expire_steps == 0) {  // nothing ever expires: only the count is reported
    if (d_n_expired) MONO_LAUNCH(prof, K_SWEEP_END, stream, sweep_nothing_kernel, dim3(1), dim3(64), d_n_expired);
    return hipGetLastError();
  }
  const uint64_t small = (2 * t.n_buckets + 256 * kSweepSmallWaves - 1) / (256 * kSweepSmallWaves);
  if (!d_expired_keys && small <= kSweepSmallBlocks) {
    MONO_LAUNCH(prof, K_SWEEP, stream, sweep_small_kernel, dim3((unsigned)small), dim3(kSweepSmallThreads), t, now, look_all,
                d_n_expired);
    return hipGetLastError();
  }
  const uint64_t waves = (2 * t.n_buckets + sweep_wave_buckets(t.capacity) - 1) / sweep_wave_buckets(t.capacity);
  const dim3 block(256), grid((unsigned)(waves < 4 * kSweepBlocks ? (waves + 3) / 4 : kSweepBlocks));
  const int keep_slots = d_expired_keys != nullptr;
  if (t.capacity >= kSweepLargeTable)
    MONO_LAUNCH(prof, K_SWEEP, stream, sweep_find_kernel<4>, grid, block, t, now, look_all, keep_slots, d_expired_keys,
                max_expired);
  else
    MONO_LAUNCH(prof, K_SWEEP, stream, sweep_find_kernel<1>, grid, block, t, now, look_all, keep_slots, d_expired_keys,
                max_expired);
  MONO_LAUNCH(prof, K_SWEEP_REMOVE, stream, sweep_remove_kernel, dim3(grid.x < 1024u ? grid.x : 1024u), block, t, now,
              d_expired_keys, max_expired, d_n_expired);
  return hipGetLastError();
}

// ---- dump --------------------------------------------------------------------------------------

__global__ void export_begin_kernel(TableView t) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  t.ctl->scratch[kExportCount] = 0;
  t.ctl->scratch[kExportBits] = 0;
  t.ctl->scratch[kExportBits + 1] = ~0ull;
}

// A block appends what it has found by one atomic, and those of all blocks meet at one word, ~12 ns each: a thread looks at
// eight slots, whose words are in flight together (a delta of 42 K keys from 2^22 slots, us: one slot 33, eight 21).
constexpr int kExportBlock = 1024, kExportPer = 8;

// touched_only: keep only the keys whose row was trained in the current synchronisation window
__global__ __launch_bounds__(kExportBlock) void export_kernel(TableView t, int64_t* keys, int32_t* rows,
                                                              uint32_t* last_seen, int64_t* slot, uint64_t max_n,
                                                              bool touched_only) {
  const uint64_t g0 = (uint64_t)blockIdx.x * (kExportBlock * kExportPer) + threadIdx.x;
  const uint32_t in_stash = t.ctl->stash_n < kStashCap ? t.ctl->stash_n : kStashCap;
  unsigned long long meta[kExportPer];
  uint32_t touch[kExportPer];
  bool live[kExportPer];
#pragma unroll
  for (int j = 0; j < kExportPer; ++j) {  // (element g: slot g, or entry g - capacity of the stash)
    const uint64_t g = g0 + (uint64_t)j * kExportBlock;
    meta[j] = g < t.capacity ? t.buckets[g >> 3].meta[g & 7] : kNoMeta;
  }
#pragma unroll
  for (int j = 0; j < kExportPer; ++j) {
    const uint64_t g = g0 + (uint64_t)j * kExportBlock;
    if (g >= t.capacity && g - t.capacity < in_stash) {
      const StashEntry& e = t.stash[g - t.capacity];
      meta[j] = make_meta(e.row, e.seen);
    }
    live[j] = meta_row(meta[j]) != kNoRow;
    touch[j] = touched_only && live[j] ? t.state[meta_row(meta[j])].touch : t.sync_epoch;
  }
  __shared__ uint32_t wave_cnt[kExportBlock / 64];
  __shared__ unsigned long long block_base;
  const uint32_t wave = threadIdx.x >> 6;
  uint64_t found[kExportPer];
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < kExportPer; ++j) {
    live[j] = live[j] && touch[j] == t.sync_epoch;
    found[j] = __ballot(live[j]);
    mine += (uint32_t)__popcll(found[j]);
  }
  if (lane_id() == 0) wave_cnt[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t all = 0;
    for (int w = 0; w < kExportBlock / 64; ++w) all += wave_cnt[w];
    block_base = all ? atomicAdd(&t.ctl->scratch[kExportCount], (unsigned long long)all) : 0ull;
  }
  __syncthreads();
  uint64_t o0 = block_base;
  for (uint32_t w = 0; w < wave; ++w) o0 += wave_cnt[w];
#pragma unroll
  for (int j = 0; j < kExportPer; ++j) {
    const uint64_t g = g0 + (uint64_t)j * kExportBlock, o = o0 + (uint64_t)__popcll(found[j] & lanes_below());
    o0 += (uint64_t)__popcll(found[j]);
    if (live[j] && o < max_n) {  // (a delta export skips most of the keys' half of the table)
      const bool in_slot = g < t.capacity;
      if (keys) keys[o] = (int64_t)(in_slot ? t.buckets[g >> 3].key[g & 7] : t.stash[g - t.capacity].key);
      if (rows) rows[o] = (int32_t)meta_row(meta[j]);
      if (last_seen) last_seen[o] = meta_seen(meta[j]);
      if (slot) slot[o] = in_slot ? (int64_t)g : -2;
    }
  }
}

hipError_t launch_export(const TableView& t, int64_t* d_keys, int32_t* d_row, uint32_t* d_last_seen, int64_t* d_slot,
                         uint64_t max_n, bool touched_only, hipStream_t stream) {
  hipLaunchKernelGGL(export_begin_kernel, dim3(1), dim3(64), 0, stream, t);
  const uint64_t total = t.capacity + kStashCap;
  constexpr uint64_t kPerBlock = kExportBlock * kExportPer;
  hipLaunchKernelGGL(export_kernel, dim3((unsigned)((total + kPerBlock - 1) / kPerBlock)), dim3(kExportBlock), 0, stream, t, d_keys,
                     d_row, d_last_seen, d_slot, max_n, touched_only);
  return hipGetLastError();
}

// A group of lanes (dim / 4 rounded up to a power of two) copies one row, four elements per lane.
template <typename E>
__global__ __launch_bounds__(256) void export_values_kernel(TableView t, const int32_t* rows, uint64_t n, float* values,
                                                            float* acc, uint32_t group_log2) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t i = g >> group_log2;
  const uint32_t l = (uint32_t)g & ((1u << group_log2) - 1u);
  if (i >= n || l * 4 >= t.dim) return;
  const uint32_t r = (uint32_t)rows[i];
  const E* src = reinterpret_cast<const E*>(t.rows) + (uint64_t)r * t.dim + l * 4;
  if (values) {
    float4 v;
    if constexpr (sizeof(E) == 2) {
      const uint2 u = *reinterpret_cast<const uint2*>(src);
      v = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                      __uint_as_float(u.y & 0xFFFF0000u));
    } else {
      v = *reinterpret_cast<const float4*>(src);
    }
    *reinterpret_cast<float4*>(values + i * t.dim + l * 4) = v;
  }
  if (acc && l == 0) acc[i] = t.state[r].acc;
}

hipError_t launch_export_values(const TableView& t, const int32_t* d_row, uint64_t n, float* d_values, float* d_acc,
                                hipStream_t stream) {
  if (n == 0) return hipSuccess;
  uint32_t group_log2 = 0;
  while ((4u << group_log2) < t.dim) ++group_log2;
  const uint64_t total = n << group_log2;
  dim3 block(256), grid((unsigned)((total + 255) / 256));
  if (t.bf16)
    hipLaunchKernelGGL(export_values_kernel<uint16_t>, grid, block, 0, stream, t, d_row, n, d_values, d_acc, group_log2);
  else
    hipLaunchKernelGGL(export_values_kernel<float>, grid, block, 0, stream, t, d_row, n, d_values, d_acc, group_log2);
  return hipGetLastError();
}

// The bus bounds it where there is much to copy (52 GB/s), and its launch where there is little: with a copy of the runtime's
// for each of the four arrays a training step of 415 IDs with its delta export took 180 us, so 128, of 42 K IDs 541 and 502.
constexpr int kCopyBlock = 256;
constexpr uint64_t kCopyBlocks = 64;  // more do not make the bus faster
__global__ __launch_bounds__(kCopyBlock) void copy_to_host_kernel(CopyParts parts, uint32_t n) {
  const uint64_t me = (uint64_t)blockIdx.x * kCopyBlock + threadIdx.x, threads = (uint64_t)gridDim.x * kCopyBlock;
  for (uint32_t p = 0; p < n; ++p) {
    const uint4* __restrict__ from = reinterpret_cast<const uint4*>(parts.from[p]);
    uint4* __restrict__ to = reinterpret_cast<uint4*>(parts.to[p]);
    const uint64_t words = parts.words[p], quads = words / 4;
    for (uint64_t i = me; i < quads; i += threads) to[i] = from[i];
    const uint64_t rest = 4 * quads + me;
    if (rest < words) reinterpret_cast<uint32_t*>(to)[rest] = reinterpret_cast<const uint32_t*>(from)[rest];
  }
}

hipError_t launch_copy_to_host(const CopyParts& parts, uint32_t n, hipStream_t stream) {
  uint64_t most = 0;
  for (uint32_t p = 0; p < n; ++p) most = parts.words[p] > most ? parts.words[p] : most;
  if (most == 0) return hipSuccess;
  const uint64_t blocks = (most + 4 * kCopyBlock - 1) / (4 * kCopyBlock);
  hipLaunchKernelGGL(copy_to_host_kernel, dim3((unsigned)(blocks < kCopyBlocks ? blocks : kCopyBlocks)), dim3(kCopyBlock), 0,
                     stream, parts, n);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void filter_export_kernel(TableView t, uint32_t* words, uint64_t first,
                                                            uint64_t count) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= count) return;
  const unsigned long long w = t.filter[first + g];
  const uint32_t cnt = (uint32_t)w > 255u ? 255u : (uint32_t)w;
  words[g] = (((uint32_t)(w >> 32) & 0xFFFFFFu) << 8) | cnt;
}

hipError_t launch_filter_export(const TableView& t, uint32_t* d_words, uint64_t first, uint64_t count,
                                hipStream_t stream) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(filter_export_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, t, d_words,
                     first, count);
  return hipGetLastError();
}

// See launch_filter_cut.  Two counters per lane, 16 bytes; the few that are too large are written.
__global__ __launch_bounds__(256) void filter_cut_kernel(TableView t) {
  const uint64_t g = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * 2;
  if (g >= t.n_filter) return;
  const uint4 w = *reinterpret_cast<const uint4*>(t.filter + g);
  if (w.x > 255u) reinterpret_cast<uint32_t*>(t.filter + g)[0] = 255u;
  if (w.z > 255u) reinterpret_cast<uint32_t*>(t.filter + g)[2] = 255u;
}

hipError_t launch_filter_cut(const TableView& t, hipStream_t stream) {
  hipLaunchKernelGGL(filter_cut_kernel, dim3((unsigned)((t.n_filter + 511) / 512)), dim3(256), 0, stream, t);
  return hipGetLastError();
}

// canonical word -> the table's own form (step << 32 | count)
__global__ __launch_bounds__(256) void filter_import_kernel(TableView t, const uint32_t* words, uint64_t first,
                                                            uint64_t count) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= count) return;
  const uint32_t w = words[g];
  t.filter[first + g] = ((unsigned long long)(w >> 8) << 32) | (unsigned long long)(w & 255u);
}

// Tables that never expire keys: a stored key stays counted.  Each of its counters inside
// [first, first + count) that the import left below the admission threshold is raised to it (a lookup
// of such a table reads a counter below the threshold as proof that the key is absent).  One thread
// per slot, then the stash.
__global__ __launch_bounds__(256) void filter_raise_kernel(TableView t, uint64_t first, uint64_t count) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint64_t key = kEmptyKey;
  if (g < t.capacity) {
    const Bucket* b = &t.buckets[g >> 3];
    if (meta_row(b->meta[g & 7]) != kNoRow) key = b->key[g & 7];
  } else if (g < t.capacity + kStashCap) {
    const uint32_t s = (uint32_t)(g - t.capacity);
    const uint32_t sn = t.ctl->stash_n < kStashCap ? t.ctl->stash_n : kStashCap;
    if (s < sn) key = t.stash[s].key;
  }
  if (key == kEmptyKey) return;
  const uint32_t least = t.freq_threshold > 1u ? t.freq_threshold : 1u;
  for (uint32_t j = 0; j < t.filter_hashes; ++j) {
    const uint64_t i = filter_index(t, key, j);
    if (i >= first && i - first < count) atomicMax(reinterpret_cast<uint32_t*>(&t.filter[i]), least);
  }
}

hipError_t launch_filter_import(const TableView& t, const uint32_t* d_words, uint64_t first, uint64_t count,
                                hipStream_t stream) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(filter_import_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, t, d_words,
                     first, count);
  if (t.expire_steps == 0) {  // (counters that age prove nothing about stored keys and stay as written)
    const uint64_t total = t.capacity + kStashCap;
    hipLaunchKernelGGL(filter_raise_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, t, first, count);
  }
  return hipGetLastError();
}

// ---- initialisation ------------------------------------------------------------------------------

// Free stack filled so that rows are handed out in ascending order: keys admitted early (the
// frequent ones) end up next to each other in memory.
__global__ __launch_bounds__(256) void init_free_rows_kernel(TableView t) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < t.capacity) t.free_rows[g] = (uint32_t)(t.capacity - 1 - g);
  if (g == 0) t.ctl->free_n = (int32_t)t.capacity;
}

hipError_t launch_table_init(const TableView& t, uint64_t dset_size, hipStream_t stream) {
  hipError_t e;
  if ((e = hipMemsetAsync(t.buckets, 0xFF, 2 * t.n_buckets * sizeof(Bucket), stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.filter, 0, t.n_filter * sizeof(unsigned long long), stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.ctl, 0, sizeof(Control), stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.win_cnt, 0, kWinLists * kWinStride * sizeof(uint32_t), stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.sweep_cnt, 0, kWinLists * kWinStride * sizeof(uint32_t), stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.oldest, 0xFF, (2 * t.n_buckets + 15) & ~15ull, stream)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(t.occupied, 0, occupancy_words(t.capacity) * sizeof(unsigned long long), stream)) != hipSuccess)
    return e;
  if ((e = hipMemsetAsync(t.dset, 0, dset_size * sizeof(unsigned long long), stream)) != hipSuccess) return e;
  hipLaunchKernelGGL(init_free_rows_kernel, dim3((unsigned)((t.capacity + 255) / 256)), dim3(256), 0, stream, t);
  return hipGetLastError();
}

}  // namespace mono
