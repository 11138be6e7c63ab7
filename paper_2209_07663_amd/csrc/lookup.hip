// lookup_or_insert: cuckoo probe, count-before-admit, insertion with bounded eviction chain,
// resolve (paper section 2.1; batch semantics of the build's contract).
//
// Three kernels per call, four where it is large (small batches have one kernel of their own: lookup_small.hip):
//   probe_count   (thread per occurrence) hit -> row index + last-seen stamp; miss -> touch the
//                 key's occurrence counter
//   admit_elect   (thread per occurrence, after ALL counts) miss with counter >= threshold -> one
//                 occurrence per distinct key is elected through the per-call dedup set and appended
//                 to one of kWinLists lists (one atomic per block, spread over the lists: a single
//                 append counter would serialise at ~12 ns per atomic on this machine)
//   insert        (dense, grid-stride over the elected occurrences) if all of them fit under the
//                 table's fill limit (else none is placed): take a row from the free stack by rank
//                 (no atomics), insert the key (CAS on 64-bit key slots, eviction chain), note it
//                 in its bucket's bound for the sweep, initialise the row with the whole wave
//   resolve       duplicates of an admitted key pick up its row, the counters are settled and the high-water mark of
//                 rows is reported to the host (in batches of at most kElectSmall by insert, beside the placement)
//
// The same kernels restore snapshot records (RestoreSource): every record is a forced
// admission whose row, accumulator and last-seen step come from the caller instead of from
// init(seed, key) / the current step; a record whose key is already stored is refused.  The
// migrate kernel re-inserts every stored element of one table into another (rehash / grow).
#include "common.h"
#include "kernels.h"
#include "table_ops.h"

namespace mono {

// The value of lane R of the quad, in all of its lanes; the value of the lane whose number differs by X (1 or 2, xor).
// (Moves inside a quad are operands of vector instructions; a shuffle goes through LDS.)
template <int R>
__device__ inline uint32_t quad_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, R * 0x55, 0xF, 0xF, true);
}
template <int X>
__device__ inline uint32_t quad_xor(uint32_t v) {
  static_assert(X == 1 || X == 2, "quad_perm 1,0,3,2 or 2,3,0,1");
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}

// Cooperative probe.  A lane owns one key; the four lanes of a quad visit the quad's four buckets one after another, and a
// lane reads two keys of the bucket (16 bytes) and their two meta words: a bucket line (eight keys, eight meta words) is two
// 64-byte accesses side by side, and the lane that finds the key has its row and stamp at hand.  The eight loads of a lane
// are independent and in flight together.
// Called by whole waves.  The bucket is looked at where `want`; found: the row, and kProbeFound | the slot, with
// kProbeStamp if its last-seen step is not `step`; else 0.
constexpr uint32_t kProbeStamp = 8, kProbeFound = 16;
struct ProbePiece {
  uint64_t key[2];
  uint32_t row[2], seen[2];
};
template <int R>
__device__ inline void probe_load(const TableView& t, uint32_t bucket, uint32_t q, ProbePiece& d) {
  const uint32_t b = quad_lane<R>(bucket);
  if (b != kNoRow) {
    const ulonglong2* line = reinterpret_cast<const ulonglong2*>(t.buckets + b);
    const ulonglong2 key = line[q];
    const uint4 meta = reinterpret_cast<const uint4*>(line)[4 + q];
    d.key[0] = key.x;
    d.key[1] = key.y;
    d.row[0] = meta.x;
    d.seen[0] = meta.y;
    d.row[1] = meta.z;
    d.seen[1] = meta.w;
  }
}
template <int R>
__device__ inline void probe_match(uint64_t k, uint32_t q, uint32_t step, const ProbePiece& d, uint32_t& row, uint32_t& found) {
  const uint64_t kr = (uint64_t)quad_lane<R>((uint32_t)(k >> 32)) << 32 | quad_lane<R>((uint32_t)k);
  const bool hit0 = d.key[0] == kr, hit1 = d.key[1] == kr;
  row = hit0 ? d.row[0] : (hit1 ? d.row[1] : 0u);
  const uint32_t seen = hit0 ? d.seen[0] : d.seen[1];
  const uint32_t code = (kProbeFound | 2 * q) + (hit1 ? 1u : 0u) + (seen != step ? kProbeStamp : 0u);
  found |= (hit0 || hit1 ? code : 0u) << (8 * R);
}
struct QuadBuckets {
  ProbePiece d[4] = {};
};
__device__ inline void probe_ask(const TableView& t, uint64_t bucket, bool want, QuadBuckets& x) {
  const uint32_t q = lane_id() & 3u, b = want ? (uint32_t)bucket : kNoRow;  // (buckets: at most 2^28)
  probe_load<0>(t, b, q, x.d[0]);
  probe_load<1>(t, b, q, x.d[1]);
  probe_load<2>(t, b, q, x.d[2]);
  probe_load<3>(t, b, q, x.d[3]);
}
__device__ inline uint32_t probe_find(uint64_t k, bool want, uint32_t step, const QuadBuckets& x, uint32_t* row_out) {
  const uint32_t q = lane_id() & 3u;
  const ProbePiece(&d)[4] = x.d;
  uint32_t row[4], found = 0;
  probe_match<0>(k, q, step, d[0], row[0], found);
  probe_match<1>(k, q, step, d[1], row[1], found);
  probe_match<2>(k, q, step, d[2], row[2], found);
  probe_match<3>(k, q, step, d[3], row[3], found);
  // at most one lane of the quad has found key r: lane r takes the words that the four have for it, together
  found |= quad_xor<1>(found);
  found |= quad_xor<2>(found);
  const bool odd = q & 1u, high = q & 2u;
  const uint32_t low01 = (odd ? row[1] : row[0]) | quad_xor<1>(odd ? row[0] : row[1]);
  const uint32_t low23 = (odd ? row[3] : row[2]) | quad_xor<1>(odd ? row[2] : row[3]);
  *row_out = (high ? low23 : low01) | quad_xor<2>(high ? low01 : low23);
  return want ? (found >> (8 * q)) & 0xFFu : 0u;
}

// Threads (= keys of a turn) per block of probe_count.  The block's missing keys are gathered in an LDS set with
// their multiplicities and each distinct one touches its counter once: a hot ID that is not (yet) admitted
// would otherwise hit one counter word with 10^5 atomics, which serialise at ~12 ns each.  The more keys a block
// takes, the fewer touches such a key makes (one per block that holds it), but a block lives as long as its
// slowest wave, and large blocks whose waves wait for each other leave the memory idle.
//   Tables that never expire keys take one turn: a key misses only until it is admitted, so hot missing keys are
//   rare after the first steps.
//   On tables with expiry counters age and the hot set may drift: every step brings hot IDs that are new.  A
//   block takes up to kProbeMaxTurns turns, one after the other without a barrier, as many as leave about
//   kProbeBlocksWanted blocks.  The set then has room for the missing keys of two turns: a hot key finds its
//   slot in the first of them; a key that finds the set full touches its counter itself.
//   (Blocks of 1024 threads that met at a barrier after two turns: 329 us per launch of 6.8 M keys where few missing
//   keys are hot, 228 us now, 272 with sixteen turns; 372 -> 349 us, 325 with sixteen, where the hot set drifts.)
constexpr int kProbeBlock = 256;
constexpr uint64_t kProbeBlocksWanted = 1024, kProbeMaxTurns = 8;
// Largest batch for which both buckets and the counter are asked for at once.  lookup_or_insert of uniform keys in a table of
// 2^24 slots, one access after the other and at once, us: a third unknown and kept out, counters that age 20 K 15.1 / 11.8, 60 K
// 16.3 / 14.4, 120 K 18.2 / 20.3, that do not 60 K 16.4 / 14.4, 120 K 19.2 / 18.4, 200 K 25.0 / 26.1; all known 20 K 8.8 / 9.0,
// 60 K 12.5 / 13.0, 120 K 14.0 / 15.9, 200 K 16.2 / 22.4.  (The rule does not ask whether the call before missed.  With a
// word for that, which the insertion writes, the three kernels of 5 K, 20 K and 60 K keys take, now and so, all known 9.9 / 9.7,
// 10.2 / 10.0, 11.2 / 10.5, of a call whose launches take the host 12 us, a third unknown 18.8 / 18.8, 19.3 / 19.5, 21.1 / 21.2, where
// counters age 18.5 / 18.8, 19.5 / 19.7, 21.1 / 21.6.)
constexpr uint64_t kProbeSmall = 1u << 16;
static_assert(kProbeSmall < 2 * kProbeBlock * kProbeBlocksWanted, "a key per thread");
constexpr int kProbeTries = 8;  // slots of the set that a missing key looks at

// restore != 0: the keys are snapshot records; a stored key is marked absent (its record is refused)
// and nothing is stamped or counted.
// A block owns kProbeBlock * turns consecutive keys and takes them in turns of one key per thread.
// kSmall (batches of at most kProbeSmall): the kernel is a chain of dependent accesses and has no bandwidth to save, so that
// both buckets, and the counter of a key that turns out to miss, are asked for at once.
// Others keep to eight waves a SIMD: a few scalar registers more left the kernel of many turns with seven (6.8 M keys 178 ->
// 172 us).
template <bool kManyTurns, bool kSmall>
__global__ __launch_bounds__(kProbeBlock, kSmall ? 1 : 8) void probe_count_kernel(TableView t,
                                                                  const int64_t* __restrict__ keys, uint64_t n, uint32_t step,
                                                                  int32_t* __restrict__ rows_out, int restore,
                                                                  uint32_t turns_, uint32_t epoch) {
  constexpr int kMissSlots = (kManyTurns ? 4 : 2) * kProbeBlock;  // slots of the block's LDS set of missing keys
  const uint32_t turns = kManyTurns ? turns_ : 1u;
  __shared__ unsigned long long miss_key[kMissSlots];
  __shared__ uint32_t miss_cnt[kMissSlots];
  // what the first counter of a missing key held, where it was looked at (see touch_word)
  constexpr bool kHolds = !kManyTurns && !kSmall;
  __shared__ unsigned long long miss_held[kHolds ? kMissSlots : 1];
  __shared__ int any_miss;
  // Are counters worth a look before the buckets?  (Counters that age prove nothing; see MissSample.)
  const bool counters_first = t.expire_steps == 0 && !restore && t.ctl->scratch[kCountersFirst] != 0;
  static_assert(!(kSmall && kManyTurns), "a small batch has a key per thread");
  const uint64_t at = (uint64_t)blockIdx.x * kProbeBlock + threadIdx.x;
  // (kSmall) the thread's key, the place in the set that it was the first to take, or none, and its counter as it was before
  const uint64_t first_key = kSmall && at < n ? (uint64_t)keys[at] : kEmptyKey;
  uint32_t first_at = kMissSlots;
  unsigned long long first_held = 0;
  const bool marks = kHolds && marks_reached(t, n);
  if (blockIdx.x == 0 && threadIdx.x < kWinLists) {  // for the election and the insertion
    t.win_cnt[threadIdx.x * kWinStride] = 0;
    if (threadIdx.x == 0) t.ctl->scratch[kFreeBefore] = (unsigned long long)(uint32_t)t.ctl->free_n;
  }
  if (threadIdx.x == 0) any_miss = 0;
  for (int s = threadIdx.x; s < kMissSlots; s += kProbeBlock) {
    miss_key[s] = kEmptyKey;
    miss_cnt[s] = 0;
  }
  __syncthreads();  // the LDS set is cleared
  bool sparse = false;  // (tables with expiry) less than a quarter full: the occupancy bitmap is worth a look
  if (t.expire_steps != 0) {
    const int32_t free_n = t.ctl->free_n;
    sparse = ((uint64_t)t.capacity - (uint64_t)(free_n < 0 ? 0 : free_n)) * 4 <= t.capacity;
  }
#pragma unroll 1
  for (uint32_t turn = 0; turn < turns; ++turn) {
    const uint64_t i = ((uint64_t)blockIdx.x * turns + turn) * kProbeBlock + threadIdx.x;
    const uint64_t k = kSmall ? first_key : (i < n ? (uint64_t)keys[i] : kEmptyKey);
    const bool live = k != kEmptyKey;
    // Negative lookup through the admission counters.  When nothing ages (expire_steps == 0) a
    // counter never decreases, and a stored key reached freq_threshold on its counter when it was
    // admitted: a counter below the threshold proves the key absent, and both bucket probes are saved.
    // Counts added by this very batch can only make the test err on the side of probing.
    bool maybe = live;
    unsigned long long held = 0;
    if (counters_first && live) {
      uint32_t cnt = 0xFFFFFFFFu;
      for (uint32_t j = 0; j < t.filter_hashes; ++j) {  // the key's count is the smallest of its counters
        const unsigned long long w = t.filter[filter_index(t, k, j)];
        if (j == 0) held = w;
        cnt = (uint32_t)w < cnt ? (uint32_t)w : cnt;
      }
      maybe = cnt >= (t.freq_threshold > 1u ? t.freq_threshold : 1u);
      if (kSmall) first_held = held;
    }
    const uint64_t b0 = bucket_index(t, 0, k), b1 = bucket_index(t, 1, k);
    // Where counters age nothing above could prove a key absent.  On a sparsely filled table the
    // occupancy bitmap, which is small enough to stay in the caches, often proves a bucket empty: such a
    // bucket is not read.  (Where the counters do the proving, the bitmap would only add a dependent
    // access: measured, 4 % on the step.)
    bool look0 = maybe, look1 = maybe;
    if (sparse && maybe) {
      look0 = (t.occupied[b0 >> 6] >> (b0 & 63)) & 1ull;
      look1 = (t.occupied[b1 >> 6] >> (b1 & 63)) & 1ull;
    }
    uint32_t row = 0, found = 0;
    uint64_t where = b0;
    QuadBuckets side1;
    if (kSmall) {
      QuadBuckets side0;
      probe_ask(t, b0, look0, side0);
      probe_ask(t, b1, look1, side1);
      if (t.expire_steps != 0 && live && !restore) first_held = t.filter[filter_index(t, k)];
      found = probe_find(k, look0, step, side0, &row);
    } else if (__ballot(look0)) {  // wave-uniform
      QuadBuckets side0;
      probe_ask(t, b0, look0, side0);
      found = probe_find(k, look0, step, side0, &row);
    }
    const bool again = look1 && found == 0;
    if (__ballot(again)) {  // wave-uniform
      uint32_t row1;
      if (!kSmall) probe_ask(t, b1, again, side1);
      const uint32_t found1 = probe_find(k, again, step, side1, &row1);
      if (again) {
        where = b1;
        row = row1;
        found = found1;
      }
    }
    bool miss = false;
    if (i < n) {
      if (!live) {
        rows_out[i] = kRowAbsent;
      } else if (found) {
        rows_out[i] = restore ? kRowAbsent : (int32_t)row;
        if (!restore && (found & kProbeStamp))
          reinterpret_cast<uint32_t*>(&t.buckets[where].meta[found & (kBucket - 1)])[1] = step;  // stamp
      } else {
        miss = true;
        const uint32_t sn = t.ctl->stash_n;
        if (sn) {
          const uint32_t lim = sn < kStashCap ? sn : kStashCap;
          for (uint32_t s = 0; s < lim && miss; ++s)
            if (t.stash[s].key == k) {
              rows_out[i] = restore ? kRowAbsent : (int32_t)t.stash[s].row;
              if (!restore) t.stash[s].seen = step;
              miss = false;
            }
        }
        if (miss) rows_out[i] = kRowMiss;
      }
    }
    if (miss) any_miss = 1;
    if (miss && !restore) {  // (records of a restore call are not occurrences: nothing is counted)
      uint32_t pos = (uint32_t)(mix64(k ^ t.s_dedup) >> 40) & (kMissSlots - 1);
      int tries = 0;
      for (; tries < kProbeTries; ++tries) {
        const unsigned long long old = atomicCAS(&miss_key[pos], (unsigned long long)kEmptyKey, (unsigned long long)k);
        if (kSmall && old == kEmptyKey) first_at = pos;
        if (kHolds && old == kEmptyKey) miss_held[pos] = held;
        if (old == kEmptyKey || old == k) break;
        pos = (pos + 1) & (kMissSlots - 1);
      }
      if (tries < kProbeTries)
        atomicAdd(&miss_cnt[pos], 1u);
      else
        marks ? touch_counter<true>(t, k, step, 1u, false, 0, epoch) : touch_counter<false>(t, k, step, 1u);
    }
  }
  __syncthreads();
  // (an ordinary store: it stays in the XCD's L2 until the kernel ends; atomic ones to one word from 26 K blocks took
  // 1.5 ms)
  if (threadIdx.x == 0 && any_miss) t.ctl->scratch[kMissTag] = epoch;
  if (restore || !any_miss) return;  // block-uniform
  if (kSmall) {
    if (first_at != kMissSlots)
      touch_counter<false>(t, first_key, step, miss_cnt[first_at], t.expire_steps != 0 || counters_first, first_held);
    return;
  }
  const bool known = kHolds && counters_first;
  for (int s = threadIdx.x; s < kMissSlots; s += kProbeBlock) {
    if (miss_cnt[s] == 0) continue;
    const unsigned long long held = kHolds ? miss_held[s] : 0;
    if (marks)
      touch_counter<true>(t, miss_key[s], step, miss_cnt[s], known, held, epoch);
    else
      touch_counter<false>(t, miss_key[s], step, miss_cnt[s], known, held);
  }
}

// ---- election ------------------------------------------------------------------------------------

// kPer: occurrences per thread.  Four for large batches: the kernel is a chain of dependent accesses (occurrence ->
// key -> dedup set -> exchange), and four of them side by side keep the memory busier than more blocks
// with one would; and an ID that turns hot before it is admitted is led by one occurrence per block, and all those
// leaders meet at one position of the dedup set.  One for batches of at most kElectSmall, which are short of blocks.
constexpr int kElectBlock = 256;
template <int kPer>
__global__ __launch_bounds__(kElectBlock, 8) void admit_elect_kernel(TableView t, const int64_t* __restrict__ keys,
                                                                     uint64_t n, uint32_t epoch, int32_t* rows_out,
                                                                     int restore, uint32_t sample_every) {
  constexpr int kElectSlots = 2 * kElectBlock * kPer;  // slots of a block's LDS set of missing keys
  constexpr int kElectWaves = kElectBlock / 64;
  __shared__ uint32_t wave_cnt[kElectWaves];
  __shared__ uint32_t block_base;
  // The block's occurrences of one missing key are represented by one of them (the leader): a key
  // that turns hot before it is admitted arrives here in thousands of occurrences, and each of them
  // re-reading the counter and competing for the same position of the dedup set serialised.
  // (When all have their places its keys make room for what the leaders find, kRowAbsent or the elected occurrence as
  // -occ - 3: with an array for that, and 80 registers, six blocks shared a compute unit instead of eight.  6.8 M keys, a
  // million of them new 92 -> 85 us, a million kept out 50 -> 44.)
  __shared__ unsigned long long s_key[kElectSlots];
  // A large batch without a miss ends here.  (A small one reads its occurrences at once: the tag before them is one more
  // round trip of a kernel that is hardly more than three.)
  if (kPer > 1 && t.ctl->scratch[kMissTag] != epoch) return;  // block-uniform
  const uint64_t i0 = (uint64_t)blockIdx.x * (kElectBlock * kPer) + threadIdx.x;
  bool miss[kPer];
  uint64_t k[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint64_t i = i0 + (uint64_t)j * kElectBlock;
    miss[j] = i < n && rows_out[i] == kRowMiss;
    if (kPer == 1) k[j] = i < n ? (uint64_t)keys[i] : kEmptyKey;  // (side by side with its word: latency is all that counts)
  }
  for (int s = threadIdx.x; s < kElectSlots; s += kElectBlock) s_key[s] = kEmptyKey;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (kPer > 1) k[j] = miss[j] ? (uint64_t)keys[i0 + (uint64_t)j * kElectBlock] : kEmptyKey;
  if (kPer > 1) {
    __syncthreads();
  } else if (!__syncthreads_or(miss[0])) {
    return;
  }
  bool leader[kPer];
  uint32_t ls[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    leader[j] = false;
    ls[j] = 0;
    if (miss[j]) {
      ls[j] = (uint32_t)(mix64(k[j] ^ t.s_dedup) >> 32) & (kElectSlots - 1);
      for (;;) {  // at most half of the slots are ever taken: a free slot always turns up
        const unsigned long long old = atomicCAS(&s_key[ls[j]], (unsigned long long)kEmptyKey, (unsigned long long)k[j]);
        if (old == kEmptyKey) leader[j] = true;
        if (old == kEmptyKey || old == k[j]) break;
        ls[j] = (ls[j] + 1) & (kElectSlots - 1);
      }
    }
  }
  // A snapshot record is admitted whatever its counter says, and with a threshold of 0 or 1 every
  // missing key is admissible (its count is at least 1 by now): no counter is read for either.
  // (Small batches ask for the key's position in the dedup set beside its counters.)
  bool admissible[kPer];
  unsigned long long e[kPer], old[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    e[j] = 0;
    if (kPer == 1 && leader[j]) e[j] = ld_agent(&t.dset[mix64(k[j] ^ t.s_dedup) & t.dset_mask]);
    uint32_t cnt = leader[j] ? 255u : 0u;
    if (!restore && leader[j] && t.freq_threshold > 1u) {
      bool look = true;
      for (uint32_t h = 0; kPer > 1 && marks_reached(t, n) && h < t.filter_hashes; ++h)
        look = look && t.reached[filter_index(t, k[j], h) & t.reached_mask] == reached_mark(epoch);
      if (!look) cnt = 0;
      for (uint32_t h = 0; look && h < t.filter_hashes; ++h) {  // smallest of the key's counters
        const uint32_t c = reinterpret_cast<const uint32_t*>(&t.filter[filter_index(t, k[j], h)])[0];
        cnt = c < cnt ? c : cnt;
      }
    }
    admissible[j] = leader[j] && cnt >= t.freq_threshold;
  }
  // one occurrence per distinct key wins its position of the per-call dedup set: a first look and a first exchange
  // for all of the thread's leaders together, then whatever is left to do for each
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (kPer > 1 && admissible[j]) e[j] = ld_agent(&t.dset[mix64(k[j] ^ t.s_dedup) & t.dset_mask]);
  }
  const unsigned long long tag = (unsigned long long)epoch << 32;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    old[j] = e[j];
    if (admissible[j] && (uint32_t)(e[j] >> 32) != epoch)
      old[j] = atomicCAS(&t.dset[mix64(k[j] ^ t.s_dedup) & t.dset_mask], e[j], tag | (i0 + (uint64_t)j * kElectBlock));
  }
  __syncthreads();  // all have their places in the set
  bool winner[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    winner[j] = false;
    if (!leader[j]) continue;
    const uint64_t i = i0 + (uint64_t)j * kElectBlock;
    int32_t found = kRowAbsent;
    if (admissible[j]) {
      uint64_t pos = mix64(k[j] ^ t.s_dedup) & t.dset_mask, owner = i;
      unsigned long long seen = old[j];
      winner[j] = (uint32_t)(e[j] >> 32) != epoch && old[j] == e[j];
      while (!winner[j]) {
        if ((uint32_t)(seen >> 32) == epoch) {  // someone wrote this position in this call
          owner = (uint32_t)seen;
          if ((uint64_t)keys[owner] == k[j]) break;  // duplicate of the owner
          pos = (pos + 1) & t.dset_mask;
          seen = ld_agent(&t.dset[pos]);
          continue;
        }
        const unsigned long long was = atomicCAS(&t.dset[pos], seen, tag | i);
        winner[j] = was == seen;
        if (winner[j]) owner = i;
        seen = was;
      }
      // (a second record of the same key in one restore call is refused like a stored key)
      found = restore ? kRowAbsent : -(int32_t)owner - 3;
    }
    s_key[ls[j]] = (unsigned long long)(uint32_t)found;
    if (!winner[j]) rows_out[i] = found;  // (the winner's word is written with its place in the list, or by the insertion)
  }
  __syncthreads();
  bool duplicate = false;
  uint32_t missed = 0;  // of the wave's occurrences, as MissSample counts them
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    int32_t found = kRowMiss;
    if (miss[j] && !winner[j]) {
      found = (int32_t)(uint32_t)s_key[ls[j]];
      if (!leader[j]) rows_out[i0 + (uint64_t)j * kElectBlock] = found;
      duplicate = duplicate || found <= -3;
    }
    missed += (uint32_t)__popcll(__ballot(kPer > 1 ? miss[j] : found == kRowAbsent));
  }
  if (kPer > 1 && __ballot(duplicate) && lane_id() == 0) t.ctl->scratch[kDuplicateTag] = epoch;
  // block-aggregated append to sub-list (blockIdx mod kWinLists)
  const uint32_t wave = threadIdx.x >> 6;
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) mine += (uint32_t)__popcll(__ballot(winner[j]));
  if (lane_id() == 0) wave_cnt[wave] = missed << 16 | mine;
  __syncthreads();
  const uint32_t list = blockIdx.x & (kWinLists - 1);
  if (threadIdx.x == 0) {
    uint32_t total = 0;  // (both halves: at most kElectBlock * kPer each)
    for (int w = 0; w < kElectWaves; ++w) total += wave_cnt[w];
    block_base = total & 0xFFFFu ? atomicAdd(&t.win_cnt[list * kWinStride], total & 0xFFFFu) : 0u;
    if (total & 0xFFFFu) t.ctl->scratch[kElectedTag] = epoch;  // (an ordinary store, as of kMissTag)
    if (sample_every && blockIdx.x % sample_every == 0 && total >> 16)
      atomicAdd(&t.ctl->scratch[kSampledMisses], (unsigned long long)(total >> 16));
  }
  __syncthreads();
  uint32_t p = block_base;
  for (uint32_t w = 0; w < wave; ++w) p += wave_cnt[w] & 0xFFFFu;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint64_t m = __ballot(winner[j]);
    if (winner[j]) {
      const uint32_t at = p + (uint32_t)__popcll(m & lanes_below());
      const uint64_t i = i0 + (uint64_t)j * kElectBlock;
      t.win_list[(uint64_t)list * t.win_cap + at] = Winner{k[j], (uint32_t)i, 0u};
      if (kPer == 1) rows_out[i] = kRowElected - (int32_t)at;  // (see insert_kernel)
    }
    p += (uint32_t)__popcll(m);
  }
}

// ---- insertion ---------------------------------------------------------------------------------

// Whether the next call is to look at counters first (see MissSample).
__device__ inline void note_sample(const TableView& t, uint64_t enough) {
  if (enough == 0) return;
  t.ctl->scratch[kCountersFirst] = t.ctl->scratch[kSampledMisses] >= enough;
  t.ctl->scratch[kSampledMisses] = 0;
}

// Dense over the elected occurrences: winner number w of the call takes free_rows[free_n - 1 - w].
// kAll (batches of at most kElectSmall): the duplicates of admitted keys take their rows here too.  The elected
// occurrence's word in rows_out tells its place in its sub-list until it holds the row (stored and read at agent scope: its
// block and the duplicates' run together), and the number of a winner follows from its place, so that nobody waits for
// anybody.  Nor does the thread that settles the counters, while other blocks run: it alone may touch free_n and hwm here, and
// all others know the free rows from kFreeBefore, which the call's first kernel has noted.  The kernel is a
// chain of dependent accesses, and with the duplicates after the insertion, in a pass of their own, and a block that
// finishes last and settles, it was one of ten.  A kernel of its own for duplicates and counters is a launch more, 3 us of a
// call that has no miss (steps of 5 to 200 K known IDs 23 -> 19, 30 -> 28, 64 -> 60 us).  Large batches have it: the
// winners' places are a write more per new key (6.8 M IDs, a million new: election and
// insertion 276 us, with resolve_kernel 267).
// (Two or three registers of a lane are spilled to keep to eight waves a SIMD.)
template <typename E, bool kAll>
__global__ __launch_bounds__(256, 8) void insert_kernel(TableView t, uint64_t n, uint32_t step, uint32_t epoch,
                                                        int32_t* rows_out, RestoreSource src, uint64_t enough) {
  // Keys that find both of their buckets full wait here until the block has placed the others: an eviction is a
  // dozen dependent accesses, and one lane in twenty that needs it (load 0.7) would hold up every wave.
  // (The list has room for all the keys of four rounds, after which it is worked off.)
  constexpr uint32_t kListRounds = 4, kLeastSpan = 8;
  __shared__ unsigned long long s_key[256 * kListRounds], s_meta[256 * kListRounds];
  __shared__ uint32_t s_waiting;
  if (threadIdx.x == 0) s_waiting = 0;
  __syncthreads();
  const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (t.ctl->scratch[kElectedTag] != epoch) {  // nothing to place or to settle (a duplicate needs an elected occurrence)
    if (kAll && blockIdx.x == 0 && threadIdx.x == 0) {
      if (t.hwm_mail && epoch % kPostEvery == 0) post_hwm(t, epoch, t.ctl->hwm);
      note_sample(t, enough);
    }
    return;
  }
  // (kAll) an occurrence for every thread, at the end of the grid where the others have elected ones (the launch has a thread
  // for every occurrence at least).  What is left of an earlier state of the word does no harm here.
  const uint64_t i = (uint64_t)(gridDim.x - 1 - blockIdx.x) * blockDim.x + threadIdx.x;
  int32_t mine = kRowAbsent;
  if (kAll && i < n) mine = rows_out[i];
  const uint32_t unit = src.seen ? kAgeLook : sweep_unit(step, t.sweep_q);
  // inclusive prefix of the sub-list fills, one list per lane
  const uint32_t inc = wave_sums(t.win_cnt[lane * kWinStride]), total = lane_value(inc, 63);
  const int32_t free0 = (int32_t)(uint32_t)t.ctl->scratch[kFreeBefore];
  if (kAll && blockIdx.x == 0 && threadIdx.x == 0) {
    settle_call(t, total, free0, t.ctl->hwm, epoch);
    note_sample(t, enough);
  }
  // all of the call's new keys fit under the fill limit, or none of them is placed
  const bool room = (int64_t)total <= rows_on_offer(t.capacity, free0);
  if constexpr (kAll) {
    const bool duplicate = mine <= -3 && mine > kRowElected;
    if (__ballot(duplicate)) {
      const uint64_t owner = duplicate ? (uint64_t)(-(int64_t)mine - 3) : 0;
      const int32_t o = duplicate ? ld_agent(&rows_out[owner]) : kRowAbsent;
      const uint32_t list = (uint32_t)(owner / kElectBlock) & (kWinLists - 1);  // (a block of the election appends to one)
      const uint32_t before = __shfl(inc, (int)(list > 0 ? list - 1 : 0));
      if (duplicate) {
        int32_t row = o;  // the row, or kRowAbsent, if the elected occurrence has it by now
        if (o <= kRowElected) {
          const uint32_t w = (list > 0 ? before : 0u) + (uint32_t)(kRowElected - o);
          row = room ? (int32_t)t.free_rows[free0 - 1 - (int32_t)w] : kRowAbsent;
        }
        rows_out[i] = row;
      }
    }
  }
  // How many winners a wave takes at a time: fewer than 64 where that would leave waves without any.  A new row's values
  // are hashes, 130 cycles of a wave for 64 of them, so that 64 rows of dim 128 hold one wave for 10 us while others have
  // none.  Training steps with 64 throughout and with this: 4.3 K IDs, most new, dim 128 79 -> 62 us; 26 K of dim 64
  // 69 -> 65; 690 K of dim 32 161 -> 152; 78 K of dim 16 in bf16 292 -> 283.  Less than eight is not faster.
  uint32_t span = 64;
  while (span > kLeastSpan && total <= gridDim.x * 2 * span) span >>= 1;
  uint32_t round = 0;
  for (uint32_t b0 = blockIdx.x * 4 * span; b0 < total; b0 += gridDim.x * 4 * span) {  // block-uniform
    const uint32_t w = b0 + wave * span + lane;
    const bool valid = lane < span && w < total;
    uint32_t before;
    const uint32_t list = list_holding(inc, w, b0 + wave * span, valid, &before);
    uint64_t k = 0;
    uint32_t row = kNoRow, occ = 0;
    if (valid) {
      const Winner e = t.win_list[(uint64_t)list * t.win_cap + (w - before)];
      occ = e.occ;
      k = e.key;
      if (room) row = t.free_rows[free0 - 1 - (int32_t)w];
      const int32_t found = row == kNoRow ? kRowAbsent : (int32_t)row;
      if (kAll)  // (the threads of its duplicates, in any block, may be looking for it)
        st_agent(&rows_out[e.occ], found);
      else
        rows_out[e.occ] = found;
      if (row != kNoRow) {
        const unsigned long long meta = make_meta(row, src.seen ? src.seen[e.occ] : step);
        if (!claim_free<kAll>(t, k, meta, unit)) {
          const uint32_t at = atomicAdd(&s_waiting, 1u);
          s_key[at] = k;
          s_meta[at] = meta;
        }
        if (src.values && t.expire_steps == 0) {
          // a restored key counts as seen freq_threshold times: its counters are raised to that
          // (records may come without their counters, and a counter below the threshold would
          // otherwise "prove" the key absent to the next lookup).  Counters that age prove nothing
          // and are left as they are: the restored table is then the snapshot, whatever the order
          // in which records and counter words arrive
          const uint32_t least = t.freq_threshold > 1u ? t.freq_threshold : 1u;
          for (uint32_t j = 0; j < t.filter_hashes; ++j)
            atomicMax(reinterpret_cast<uint32_t*>(&t.filter[filter_index(t, k, j)]), least);
        }
      }
    }
    init_new_rows<E>(t, valid && row != kNoRow, span, k, row, occ, src);
    if (++round == kListRounds || b0 + gridDim.x * 4 * span >= total) {
      __syncthreads();
      for (uint32_t q = threadIdx.x; q < s_waiting; q += blockDim.x) cuckoo_insert(t, s_key[q], s_meta[q], unit);
      __syncthreads();
      if (threadIdx.x == 0) s_waiting = 0;
      __syncthreads();
      round = 0;
    }
  }
}

// (large batches) Duplicates of admitted keys, and what insert_kernel settles for the others.
__global__ __launch_bounds__(256) void resolve_kernel(TableView t, uint64_t n, int32_t* rows_out, uint32_t epoch,
                                                      uint64_t enough) {
  if (t.ctl->scratch[kDuplicateTag] == epoch) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
      const int32_t v = rows_out[i];
      if (v <= -3) rows_out[i] = rows_out[-(int64_t)(v + 3)];  // (the elected occurrence has its row, or kRowAbsent, by now)
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < kWinLists) {  // (the insert kernel has finished)
    const uint32_t total = lane_value(wave_sums(t.win_cnt[threadIdx.x * kWinStride]), 63);
    if (threadIdx.x == 0) {
      settle_call(t, total, t.ctl->free_n, t.ctl->hwm, epoch);
      note_sample(t, enough);
    }
  }
}

// Records of a restore call that were refused (rows_out < 0 after the resolve step) -> scratch slot.
__global__ __launch_bounds__(256) void count_refused_kernel(TableView t, uint64_t n, const int32_t* rows_out) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t m = __ballot(i < n && rows_out[i] < 0);
  if (m && lane_id() == 0) atomicAdd(&t.ctl->scratch[kRefusedRecords], (unsigned long long)__popcll(m));
}

hipError_t launch_lookup_or_insert(const TableView& t, const int64_t* d_keys, uint64_t n, uint32_t step, uint32_t epoch,
                                   int32_t* d_rows_out, const RestoreSource& src, hipStream_t stream, Profiler* prof) {
  if (n == 0) return hipSuccess;
  const int restore = src.values != nullptr;
  if (!restore && n <= kSmallLookup) return launch_lookup_small(t, d_keys, n, step, epoch, d_rows_out, stream, prof);
  const dim3 block(256), grid((unsigned)((n + 255) / 256));
  // (insertion: a wave for 16 IDs, all of which may be new; see insert_kernel's span)
  const uint64_t iblocks = (n + 63) / 64;
  constexpr uint64_t kInsertBlocks = 2048;
  static_assert(kInsertBlocks * 256 >= kElectSmall, "a thread for every occurrence of a batch that has no resolve_kernel");
  const dim3 igrid((unsigned)(iblocks < kInsertBlocks ? iblocks : kInsertBlocks));
  {
    uint64_t turns = t.expire_steps == 0 ? 1 : n / ((uint64_t)kProbeBlock * kProbeBlocksWanted);
    turns = turns < 1 ? 1 : (turns > kProbeMaxTurns ? kProbeMaxTurns : turns);
    const uint64_t per_block = (uint64_t)kProbeBlock * turns;
    const dim3 pgrid((unsigned)((n + per_block - 1) / per_block));
    if (n <= kProbeSmall)
      MONO_LAUNCH(prof, K_PROBE_COUNT, stream, (probe_count_kernel<false, true>), pgrid, dim3(kProbeBlock), t, d_keys, n, step,
                  d_rows_out, restore, 1u, epoch);
    else if (turns == 1)
      MONO_LAUNCH(prof, K_PROBE_COUNT, stream, (probe_count_kernel<false, false>), pgrid, dim3(kProbeBlock), t, d_keys, n, step,
                  d_rows_out, restore, 1u, epoch);
    else
      MONO_LAUNCH(prof, K_PROBE_COUNT, stream, (probe_count_kernel<true, false>), pgrid, dim3(kProbeBlock), t, d_keys, n, step,
                  d_rows_out, restore, (uint32_t)turns, epoch);
  }
  const uint64_t elect_per_block = n <= kElectSmall ? kElectBlock : 4 * kElectBlock;
  const dim3 egrid((unsigned)((n + elect_per_block - 1) / elect_per_block));
  MissSample sample = {0, 0};
  if (t.expire_steps == 0 && !restore) sample = miss_sample(n, egrid.x, elect_per_block);
  if (n <= kElectSmall)
    MONO_LAUNCH(prof, K_ADMIT_ELECT, stream, admit_elect_kernel<1>, egrid, block, t, d_keys, n, epoch, d_rows_out, restore,
                sample.every);
  else
    MONO_LAUNCH(prof, K_ADMIT_ELECT, stream, admit_elect_kernel<4>, egrid, block, t, d_keys, n, epoch, d_rows_out, restore,
                sample.every);
#define MONO_INSERT(E, all) \
  MONO_LAUNCH(prof, K_INSERT, stream, (insert_kernel<E, all>), igrid, block, t, n, step, epoch, d_rows_out, src, sample.enough)
  if (n <= kElectSmall) {
    if (t.bf16)
      MONO_INSERT(uint16_t, true);
    else
      MONO_INSERT(float, true);
  } else {
    if (t.bf16)
      MONO_INSERT(uint16_t, false);
    else
      MONO_INSERT(float, false);
    MONO_LAUNCH(prof, K_RESOLVE, stream, resolve_kernel, igrid, block, t, n, d_rows_out, epoch, sample.enough);
  }
#undef MONO_INSERT
  if (restore) hipLaunchKernelGGL(count_refused_kernel, grid, block, 0, stream, t, n, d_rows_out);
  return hipGetLastError();
}

// ---- rehash / grow -------------------------------------------------------------------------------

// Every stored element of `src` (slots, then the stash) is inserted into `dst` under dst's hash
// functions, with its row index and last-seen step unchanged (the rows themselves are copied
// separately, position for position).  Elements are distinct and none is in dst: the insertion
// protocol's preconditions hold.
__global__ __launch_bounds__(256) void migrate_kernel(TableView dst, TableView src) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < src.capacity) {
    const Bucket* b = &src.buckets[g >> 3];
    const unsigned long long m = b->meta[g & 7];
    if (meta_row(m) != kNoRow) cuckoo_insert(dst, b->key[g & 7], m, kAgeLook);
  } else if (g < src.capacity + kStashCap) {
    const uint32_t s = (uint32_t)(g - src.capacity);
    const uint32_t sn = src.ctl->stash_n < kStashCap ? src.ctl->stash_n : kStashCap;
    if (s < sn) cuckoo_insert(dst, src.stash[s].key, make_meta(src.stash[s].row, src.stash[s].seen), kAgeLook);
  }
}

// Free stack of the grown table: the new rows at the bottom (handed out last, in ascending order),
// the free rows of the old table above them in their old order.
__global__ __launch_bounds__(256) void migrate_free_rows_kernel(TableView dst, TableView src, int32_t src_free_n) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t extra = dst.capacity - src.capacity;
  if (g < extra)
    dst.free_rows[g] = (uint32_t)(dst.capacity - 1 - g);
  else if (g < extra + (uint64_t)src_free_n)
    dst.free_rows[g] = src.free_rows[g - extra];
}

// Counter i of the grown array takes the value of the counter its keys used to share (top-bit
// addressing: old index = new index >> shift).
__global__ __launch_bounds__(256) void migrate_filter_kernel(TableView dst, TableView src, uint32_t shift) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < dst.n_filter) dst.filter[g] = src.filter[g >> shift];
}

hipError_t launch_migrate(const TableView& dst, const TableView& src, int32_t src_free_n, hipStream_t stream) {
  uint32_t shift = 0;
  while ((src.capacity << shift) < dst.capacity) ++shift;
  const dim3 block(256);
  hipLaunchKernelGGL(migrate_filter_kernel, dim3((unsigned)((dst.n_filter + 255) / 256)), block, 0, stream, dst, src,
                     shift);
  hipLaunchKernelGGL(migrate_free_rows_kernel, dim3((unsigned)((dst.capacity + 255) / 256)), block, 0, stream, dst, src,
                     src_free_n);
  const uint64_t total = src.capacity + kStashCap;
  hipLaunchKernelGGL(migrate_kernel, dim3((unsigned)((total + 255) / 256)), block, 0, stream, dst, src);
  return hipGetLastError();
}

}  // namespace mono
