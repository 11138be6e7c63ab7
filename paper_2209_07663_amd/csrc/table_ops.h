// Device functions that change a table: occurrence counters, insertion with its eviction chain, the initial
// state of new rows.  Shared by the kernels of lookup_or_insert, restore and migrate.
//
// Slot protocol (no 128-bit atomics, no fences): a slot's `meta` word doubles as its lock.
//   free slot:   key == EMPTY, meta == kNoMeta
//   claim:       CAS key EMPTY -> k (wait for the result); then store meta (publishes row + stamp)
//   evict:       old = exch(meta, kNoMeta); row(old) == kNoRow -> slot is free or mid-write, try
//                another; else the caller owns the slot: vk = exch(key, k) (wait), then store meta.
//                The victim (vk, old) continues in its other sub-table.
// Every access in the protocol is an agent-scope atomic performed at the coherence point, and each
// step consumes the result of the previous one, so no ordering fence is needed.  No thread ever
// waits for another one; every loop is bounded.
#pragma once

#include "common.h"
#include "kernels.h"

namespace mono {

// Are counters marked that are at the threshold (see reached_mark)?
__device__ inline bool marks_reached(const TableView& t, uint64_t n) {
  return t.expire_steps == 0 && t.freq_threshold > 1u && n > kElectSmall;
}

// Counts are kept unsaturated in the low half of a counter word and read as min(count, 255).  Where
// counters age, the first touch of a batch cuts the count back to 255; where they do not, the host has all counts cut
// back (launch_filter_cut) before they could have taken more than kCountMost occurrences since the last time.
// one counter word: `times` occurrences at `step`; `held`, if `known`: what it held a moment ago (an ordinary
// load will do, the exchange tells whether it still holds that).  kMark (where nothing ages): notes a count that is at the
// threshold now.
template <bool kMark>
__device__ inline void touch_word(const TableView& t, uint64_t at, uint32_t step, uint32_t times, bool known,
                                  unsigned long long held, uint32_t epoch) {
  unsigned long long* w = &t.filter[at];
  if (t.expire_steps == 0) {
    // nothing ever ages: the stamp only moves forward and the count only grows, so two atomics
    // whose results nobody waits for do it (low half = count, high half = last step).  Who knows what the word held needs one
    // of them only: an exchange, or the addition where the step is noted already (6.8 M keys, a fifth of them missing: the
    // probe 195 -> 186 us).
    uint32_t* half = reinterpret_cast<uint32_t*>(w);
    const bool noted = known && (uint32_t)(held >> 32) >= step;
    const unsigned long long want = ((unsigned long long)step << 32) | (uint32_t)((uint32_t)held + times);
    uint32_t now = (uint32_t)want;  // the count with these occurrences
    if (!known || noted || atomicCAS(w, held, want) != held) {
      if (!noted) atomicMax(half + 1, step);
      now = atomicAdd(half, times) + times;
    }
    if (kMark && now >= t.freq_threshold) t.reached[at & t.reached_mask] = reached_mark(epoch);
    return;
  }
  unsigned long long cur = known ? held : ld_agent(w);
  for (;;) {
    if ((uint32_t)(cur >> 32) == step) {  // already touched in this batch: increments only
      atomicAdd(w, (unsigned long long)times);  // unsaturated; read as min(count, 255)
      return;
    }
    // first toucher of the batch: ages the word, stamps the step and adds its occurrences in one exchange
    uint32_t last = (uint32_t)(cur >> 32), cnt = (uint32_t)cur;
    if (cnt > 255u) cnt = 255u;  // the unsaturated count is cut back once per batch: it can never wrap
    if (step - last >= t.expire_steps) cnt = 0;
    const unsigned long long want = ((unsigned long long)step << 32) | (unsigned long long)(cnt + times);
    const unsigned long long old = atomicCAS(w, cur, want);
    if (old == cur) return;
    cur = old;
  }
}

// every counter of the key (section 2.1's probabilistic filter read as a counting filter with
// filter_hashes hashes; two hashes of a key that fall on one counter touch it twice, as the oracle does)
template <bool kMark>
__device__ inline void touch_counter(const TableView& t, uint64_t key, uint32_t step, uint32_t times, bool known_first = false,
                                     unsigned long long held_first = 0, uint32_t epoch = 0) {
  for (uint32_t j = 0; j < t.filter_hashes; ++j)
    touch_word<kMark>(t, filter_index(t, key, j), step, times, j == 0 && known_first, held_first, epoch);
}

__device__ inline void wait_all_memory_ops() {
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);  // every load, store and atomic of this wave has been performed
  __asm__ volatile("" ::: "memory");
}

// Notes for the sweep that bucket b has taken a key (tables with expiry).  `unit`: the unit of the current step if the
// key's last-seen step is that (no key can be newer, so a bucket that holds something keeps its bound), or
// kAgeLook for a key that was seen earlier or at an unknown time.  `word`: the byte, in its word, read with an ordinary load:
// a stale copy can only show kAgeEmpty where another compute unit has noted a key in this very kernel
// (bytes become kAgeEmpty in the sweep alone, in a kernel of its own).  Bits are only ever cleared here: all who
// note the current unit write the same one, and kAgeLook wins over any.
__device__ inline void note_key(const TableView& t, const Bucket* b, uint32_t unit, uint32_t word) {
  if (t.expire_steps == 0) return;
  const uint64_t idx = (uint64_t)(b - t.buckets);
  const uint32_t at = 8u * (uint32_t)(idx & 3), have = (word >> at) & 0xFFu;
  if (have == kAgeEmpty) atomicOr(&t.occupied[idx >> 6], 1ull << (idx & 63));
  if (have == kAgeEmpty || (unit == kAgeLook && have != kAgeLook)) atomicAnd(&t.oldest[idx >> 2], (unit << at) | ~(0xFFu << at));
}
// The word of `oldest` that note_key wants, asked for before it is known whether the bucket takes the key.
__device__ inline uint32_t age_word(const TableView& t, const Bucket* b) {
  return t.expire_steps == 0 ? 0u : t.oldest[(uint64_t)(b - t.buckets) >> 2];
}

// kAtOnce: the bucket's byte is asked for with its keys, whether it is wanted or not (a small batch has no bandwidth to save).
template <bool kAtOnce = false>
__device__ inline bool try_claim(const TableView& t, Bucket* b, uint64_t k, unsigned long long meta, uint32_t unit) {
  // snapshot of the eight keys (may be stale: a slot seen free may be taken by now; the CAS decides)
  const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(b->key);
  const ulonglong2 a0 = kp[0], a1 = kp[1], a2 = kp[2], a3 = kp[3];
  uint32_t word = kAtOnce ? age_word(t, b) : 0u;
  const uint64_t snap[kBucket] = {a0.x, a0.y, a1.x, a1.y, a2.x, a2.y, a3.x, a3.y};
  uint32_t open = 0;
#pragma unroll
  for (int l = 0; l < kBucket; ++l) open |= snap[l] == kEmptyKey ? 1u << l : 0u;
  // A bucket that holds a key has its bound, or gets it from whoever placed that key in this kernel: its byte is not even
  // read, which was an eighth of what the insertion of a million keys moved (169 -> 147 us).  Else the read goes beside the
  // exchange.
  const bool note = unit == kAgeLook || open == (1u << kBucket) - 1u;
  if (!kAtOnce && note && open) word = age_word(t, b);
#pragma unroll 1
  for (; open; open &= open - 1) {
    const uint32_t l = (uint32_t)__ffs((int)open) - 1u;
    if (atomicCAS((unsigned long long*)&b->key[l], (unsigned long long)kEmptyKey, (unsigned long long)k) ==
        (unsigned long long)kEmptyKey) {
      st_agent(&b->meta[l], meta);  // issued after the CAS has returned: publishes the slot
      if (note) note_key(t, b, unit, word);
      return true;
    }
  }
  return false;
}

__device__ inline bool has_empty_key(const Bucket* b) {
  const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(b->key);
  const ulonglong2 a0 = kp[0], a1 = kp[1], a2 = kp[2], a3 = kp[3];
  return a0.x == kEmptyKey || a0.y == kEmptyKey || a1.x == kEmptyKey || a1.y == kEmptyKey || a2.x == kEmptyKey ||
         a2.y == kEmptyKey || a3.x == kEmptyKey || a3.y == kEmptyKey;
}

// Which resident of the full bucket b (in sub-table `side`) to evict.  A victim whose OTHER bucket has
// a free slot ends the chain after one move, so the other buckets of the eight residents are looked
// at first (eight independent line reads) and the first such resident from `start` on is chosen;
// if there is none, `start` itself.  Only a hint: the snapshot may be stale, the protocol decides.
// Measured on the streaming configuration at load 0.92: a random victim gave chains of up to 20
// evictions, each five dependent memory round trips long, and the slowest chain is the kernel's time.
__device__ inline uint32_t pick_victim(const TableView& t, const Bucket* b, int side, uint32_t start) {
  const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(b->key);
  const ulonglong2 a0 = kp[0], a1 = kp[1], a2 = kp[2], a3 = kp[3];
  const uint64_t res[kBucket] = {a0.x, a0.y, a1.x, a1.y, a2.x, a2.y, a3.x, a3.y};
  uint32_t good = 0;  // bit l: resident l could move out at once
#pragma unroll
  for (int l = 0; l < kBucket; ++l) {
    if (res[l] == kEmptyKey) continue;
    if (has_empty_key(&t.buckets[bucket_index(t, 1 - side, res[l])])) good |= 1u << l;
  }
  if (good == 0) return start;
  const uint32_t rotated = ((good >> start) | (good << (kBucket - start))) & 0xFFu;  // bit 0 = slot `start`
  return (start + (uint32_t)__ffs((int)rotated) - 1u) & (kBucket - 1);
}

// Takes a free slot of either bucket of k, if there is one (see cuckoo_insert).
template <bool kAtOnce>
__device__ inline bool claim_free(const TableView& t, uint64_t k, unsigned long long meta, uint32_t unit) {
  return try_claim<kAtOnce>(t, &t.buckets[bucket_index(t, 0, k)], k, meta, unit) ||
         try_claim<kAtOnce>(t, &t.buckets[bucket_index(t, 1, k)], k, meta, unit);
}

// Inserts (k, meta); k is not in the table and no other thread inserts the same key.  unit: see note_key.
__device__ void cuckoo_insert(const TableView& t, uint64_t k, unsigned long long meta, uint32_t unit) {
  int side = 0;
  uint32_t chain = 0;
#pragma unroll 1
  for (int kick = 0; kick < kMaxKicks; ++kick) {
    Bucket* b = &t.buckets[bucket_index(t, side, k)];
    if (try_claim(t, b, k, meta, unit)) goto done;
    if (kick == 0 && try_claim(t, &t.buckets[bucket_index(t, 1, k)], k, meta, unit)) goto done;
    // evict: take the lock of a published slot
    const uint32_t v0 = pick_victim(t, b, side, (uint32_t)(mix64(k + (uint64_t)kick) >> 61));
#pragma unroll 1
    for (int tries = 0; tries < kBucket; ++tries) {
      const int l = (int)((v0 + (uint32_t)tries) & (kBucket - 1));
      const unsigned long long old = atomicExch(&b->meta[l], kNoMeta);
      if (meta_row(old) == kNoRow) continue;  // free or mid-write: not ours
      const uint64_t vk = atomicExch((unsigned long long*)&b->key[l], (unsigned long long)k);
      wait_all_memory_ops();  // the key exchange is performed before the slot is published again
      st_agent(&b->meta[l], meta);
      // (a key of the current step leaves the bound of a full bucket as it is)
      if (unit == kAgeLook) note_key(t, b, unit, age_word(t, b));
      k = vk;
      meta = old;
      unit = kAgeLook;
      side = 1 - side;  // the victim continues in its other sub-table
      ++chain;
      break;
    }
  }
  {  // chain bound hit: keep the homeless element aside
    const uint32_t s = atomicAdd(&t.ctl->stash_n, 1u);
    atomicAdd(&t.ctl->n_insert_failed, 1ull);
    if (s < kStashCap) {
      t.stash[s].key = k;
      t.stash[s].row = meta_row(meta);
      t.stash[s].seen = meta_seen(meta);
    } else {
      atomicAdd(&t.ctl->n_lost, 1ull);
    }
  }
done:
  // (read first: an atomic on this one word from every insertion that evicted serialises at ~12 ns each,
  // which at load 0.8 was most of the kernel's time)
  if (chain && (unsigned long long)chain > ld_agent(&t.ctl->max_chain))
    atomicMax(&t.ctl->max_chain, (unsigned long long)chain);
}

template <typename E>
__device__ inline void store_init4(E* rows, uint64_t idx, float4 v);
template <>
__device__ inline void store_init4<float>(float* rows, uint64_t idx, float4 v) {
  *reinterpret_cast<float4*>(rows + idx) = v;
}
template <>
__device__ inline void store_init4<uint16_t>(uint16_t* rows, uint64_t idx, float4 v) {
  uint2 u;
  u.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
  u.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
  *reinterpret_cast<uint2*>(rows + idx) = u;
}

// The wave initialises its new rows together: a group of dim/4 lanes per row (at most the whole wave, which
// then walks the row in pieces of 256 elements), four elements per lane, 64/group rows at a time, stored as
// whole 16-byte (fp32) or 8-byte (bf16) pieces.  Called by a whole wave; ok: this lane, one of the first `lanes`, has a new
// row `row` for key k, `occ` is the record it comes from (src.values != nullptr) or unused.
template <typename E>
__device__ inline void init_new_rows(const TableView& t, bool ok_lane, uint32_t lanes, uint64_t k, uint32_t row, uint32_t occ,
                                     const RestoreSource& src) {
  const uint32_t lane = lane_id();
  E* rows = reinterpret_cast<E*>(t.rows);
  uint32_t glog = 0;
  while (glog < 6 && (4u << glog) < t.dim) ++glog;
  const uint32_t group = 1u << glog, per_round = 64u >> glog, l = lane & (group - 1u), gi = lane >> glog;
  if (__ballot(ok_lane) == 0) return;  // wave-uniform
  const uint64_t mine = mix64(k ^ t.s_init);
  const uint32_t row_or_none = ok_lane ? row : kNoRow;
  for (uint32_t q = 0; q * per_round < lanes; ++q) {
    const int from = (int)(q * per_round + gi);
    const uint64_t base_h = __shfl(mine, from);
    const uint32_t rr = __shfl(row_or_none, from);
    const uint32_t oo = src.values || src.acc ? __shfl(occ, from) : 0u;
    if (rr == kNoRow) continue;
    for (uint32_t col = l * 4; col < t.dim; col += 256) {
      float4 v;
      if (src.values) {
        v = *reinterpret_cast<const float4*>(src.values + (uint64_t)oo * t.dim + col);
      } else {
        v = make_float4(init_value(base_h, col), init_value(base_h, col + 1), init_value(base_h, col + 2),
                        init_value(base_h, col + 3));
      }
      store_init4<E>(rows, (uint64_t)rr * t.dim + col, v);
    }
    if (l == 0) t.state[rr] = RowState{src.acc ? src.acc[oo] : 0.0f, 0u};
  }
}

// A small call that has not moved the mark tells the host only now and then: the store over the bus holds the kernel's end.
constexpr uint32_t kPostEvery = 16;  // (far fewer than the calls that the host keeps on record)

// Tells the host the high-water mark of rows after call `epoch` (it reads the word when it pleases; the mark
// only ever grows, so a stale value is a safe one).
__device__ inline void post_hwm(const TableView& t, uint32_t epoch, uint32_t hwm) {
  __hip_atomic_store(t.hwm_mail, ((unsigned long long)epoch << 32) | (unsigned long long)hwm, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_SYSTEM);
}

// Settles the counters of a call that elected `total` new keys when free0 rows were free and the mark was hwm0.  One thread,
// when nobody reads free_n or hwm any more: after all others, or beside them where they go by kFreeBefore (insert_kernel).  It
// reads nothing itself, which would be one more trip to memory at the end.
__device__ inline void settle_call(const TableView& t, uint32_t total, int32_t free0, uint32_t hwm0, uint32_t epoch) {
  const uint32_t offer = (uint32_t)rows_on_offer(t.capacity, free0);
  const uint32_t got = total <= offer ? total : 0u;  // all of the call's new keys or none
  t.ctl->free_n = free0 - (int32_t)got;
  const uint32_t in_use = (uint32_t)t.capacity - (uint32_t)(free0 - (int32_t)got);
  if (in_use > hwm0) t.ctl->hwm = in_use;  // rows are handed out in ascending order
  if (t.hwm_mail) post_hwm(t, epoch, in_use > hwm0 ? in_use : hwm0);
  if (got) atomicAdd(&t.ctl->n_admitted, (unsigned long long)got);
  if (total - got) atomicAdd(&t.ctl->n_full, (unsigned long long)(total - got));
}

}  // namespace mono
