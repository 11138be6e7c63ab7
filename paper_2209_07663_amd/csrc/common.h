// Device-side layout and helpers shared by the kernels of the collisionless table (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace mono {

constexpr uint64_t kEmptyKey = ~0ull;       // reserved key: padding / free slot
constexpr uint32_t kNoRow = 0xFFFFFFFFu;    // slot has no published row: free, or being written
constexpr int kBucket = 8;                  // slots per bucket
constexpr int kMaxKicks = 512;              // bound of an eviction chain
constexpr int kReserveShift = 5;            // capacity >> 5 rows are never handed out: see rows_on_offer()
constexpr uint32_t kStashCap = 4096;        // homeless elements kept aside after a failed chain
constexpr int32_t kRowAbsent = -1;          // rows_out: key not in the table
constexpr int32_t kRowMiss = -2;            // rows_out, between the kernels of one call: missed, undecided
// rows_out values <= -3 between the kernels of one call: duplicate of an admitted key, -occ - 3 of the occurrence
// that was elected for it; (batches of at most kElectSmall) of that occurrence, kRowElected - its place in its sub-list
constexpr int32_t kRowElected = -(1 << 29);  // (a batch has at most 2^28 occurrences)

// One bucket = one 128-byte line (the unit the memory system fetches): eight keys, then eight
// `meta` words = last-seen step << 32 | row index.  A probe costs one line per bucket; the row and
// the stamp of a hit sit in the line already fetched.  meta == kNoMeta: slot free or being written.
struct __attribute__((aligned(128))) Bucket {
  uint64_t key[kBucket];
  unsigned long long meta[kBucket];
};
static_assert(sizeof(Bucket) == 128, "bucket must be one 128-byte line");
constexpr unsigned long long kNoMeta = ~0ull;
__host__ __device__ inline uint32_t meta_row(unsigned long long m) { return (uint32_t)m; }
__host__ __device__ inline uint32_t meta_seen(unsigned long long m) { return (uint32_t)(m >> 32); }
__host__ __device__ inline unsigned long long make_meta(uint32_t row, uint32_t seen) {
  return ((unsigned long long)seen << 32) | row;
}
constexpr int kWinLists = 64;               // sub-lists of elected occurrences (spreads the append counter)
constexpr int kWinStride = 32;              // u32 words between two sub-list counters (one 128-byte line each)

constexpr int kSweepRemoved = 0;            // Control::scratch slot: keys removed so far by the running sweep
constexpr int kExportCount = 1;             // Control::scratch slot: elements found by the running export
constexpr int kExportBits = 9;              // Control::scratch slots (two): OR and AND of the keys it found
constexpr int kValidPairs = 2;              // Control::scratch slot: (row, bag) pairs kept by the sort
constexpr int kRefusedRecords = 3;          // Control::scratch slot: records refused by the running restore call

constexpr int kSmallMisses = 4;             // Control::scratch slots of the one-kernel lookup: missing occurrences so far, blocks
constexpr int kSmallDone = 5;               // that have finished their probes and their misses (zero between calls);
constexpr int kSmallGo = 15;                // tag << 32 | number of new rows, of the latest such call with misses; the next
constexpr int kSmallNext = 16;              // chunk of them that nobody has taken yet
constexpr int kOrderDone = 17;              // Control::scratch slots: blocks of order_tiles that are done, and their tiles of one
constexpr int kOrdered = 18;                // row (zero between calls); 1 + tiles of several rows if seg_reduce is to take that order
constexpr int kMissTag = 7;                 // Control::scratch slots: tag of the latest call in which an occurrence missed,
constexpr int kDuplicateTag = 8;            // and of the latest one that has duplicates of admitted keys to resolve
constexpr int kElectedTag = 19;             // Control::scratch slot: tag of the latest call in which an occurrence was elected
constexpr int kSampledMisses = 11;          // Control::scratch slots: missing occurrences in the running call's sample (see
constexpr int kCountersFirst = 12;          // MissSample); is the next call to look at counters before buckets?
constexpr int kFreeBefore = 14;             // Control::scratch slot: rows that were free when the running call began (free_n itself
                                            // may be settled by one thread of insert_kernel while the others run)
constexpr int kHotBins = 13;                // Control::scratch slot: rows with a bin of their own (see sort_split.hip)
constexpr int kSweepDone = 6;               // Control::scratch slot: sub-lists, or blocks, that are done; of sweep_small also the keys
                                            // removed so far << 32 (zero between calls)

struct StashEntry {
  uint64_t key;
  uint32_t row;
  uint32_t seen;
};

// Per-row optimizer state.  `touch` is the number of the synchronisation window in which the row
// was last trained (paper section 2.2.3: touched keys); it shares the accumulator's 8-byte word so
// that marking a row costs no memory access of its own.
struct alignas(8) RowState {
  float acc;
  uint32_t touch;
};

// An elected occurrence: its key travels with it, so that the insertion reads the list and nothing else.
struct alignas(16) Winner {
  uint64_t key;
  uint32_t occ;   // occurrence index in the batch
  uint32_t pad;
};

// Counters that live on the device for the whole life of the table.
struct Control {
  int32_t free_n;            // rows on the free stack
  uint32_t stash_n;          // elements pushed to the stash (may exceed kStashCap: then some were lost)
  uint32_t hwm;              // every row index ever handed out is below this high-water mark
  uint32_t swept;            // step of the latest sweep
  unsigned long long n_admitted, n_expired, n_insert_failed, n_lost, n_full, max_chain;
  unsigned long long scratch[20];  // per-call scalars, indexed by the constants above
};

// Everything a kernel needs to know about a table; passed by value.
struct TableView {
  Bucket* buckets;           // [2 * n_buckets]: T0 then T1
  unsigned long long* filter;  // [n_filter] occurrence counters: step << 32 | count
  void* rows;                // [capacity * dim] fp32 or bf16
  RowState* state;           // [capacity] Adagrad accumulator + touched mark
  uint32_t* free_rows;       // [capacity] stack of free row indices
  Control* ctl;
  StashEntry* stash;         // [kStashCap]
  unsigned long long* dset;  // [dset_size] per-call dedup set: epoch << 32 | occurrence index
  Winner* win_list;          // [kWinLists * win_cap] elected occurrences
  uint32_t* win_cnt;         // [kWinLists * kWinStride] fill of each sub-list (the call's first kernel clears them)
  uint64_t win_cap;
  // (tables with expiry) per bucket, for the sweep: a lower bound of the last-seen steps of its keys, in units of
  // 1 << sweep_q steps (see sweep_unit); kAgeEmpty: the bucket holds nothing; kAgeLook: nothing is known.
  // One bit per bucket beside it, set while the byte is not kAgeEmpty: small enough to stay in the caches
  // of a probe.
  uint32_t* oldest;          // [2 * n_buckets] bytes, handled as words
  unsigned long long* occupied;  // [capacity / 512, at least 1]
  uint32_t* sweep_list;      // [kWinLists * sweep_cap] rows (or slots) of the keys that the running sweep removes
  uint32_t* sweep_cnt;       // [kWinLists * kWinStride] fill of each sub-list, and in the word beside it the blocks that are
                             // done with it (all zero between calls)
  uint64_t sweep_cap;
  uint8_t* reached;          // [reached_mask + 1] per counter (by the low bits of its index): mark of the latest large call
  uint64_t reached_mask;     // in which one with these bits was at the threshold (see reached_mark)
  uint64_t capacity;
  uint64_t n_buckets;        // per sub-table
  uint64_t n_filter;
  uint64_t dset_mask;
  uint64_t s_h0, s_h1, s_init, s_dedup;
  uint64_t s_filter[4];      // one salt per counter hash
  uint32_t bucket_shift;     // 64 - log2(n_buckets)   (64 means: single bucket)
  uint32_t filter_shift;     // 64 - log2(n_filter)
  uint32_t dim;
  uint32_t freq_threshold;
  uint32_t expire_steps;
  uint32_t sweep_q;          // log2 of the unit of `oldest`, so that expire_steps are at most kAgeUnits of them
  uint32_t bf16;
  uint32_t filter_hashes;    // counters per key (1..4); the key's count is their minimum
  uint32_t sync_epoch;       // current synchronisation window (>= 1); rows with touch == sync_epoch are "touched"
  unsigned long long* hwm_mail;  // pinned HOST word (or null): lookup_or_insert leaves (its call tag << 32 | hwm)
                                 // there, so that the host can bound the sort's key width without waiting
};

__host__ __device__ inline uint64_t mix64(uint64_t z) {
  z ^= z >> 30;
  z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27;
  z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}

// Rows that new keys may take when free_n rows are free.  The last 1/32 of the rows is held back:
// with buckets of eight slots, eviction chains grow steeply past a load of ~0.97 (measured: chains
// of 125 evictions at 0.965), and a chain that hits its bound costs a stash entry, then a resident.
// A table therefore stores at most capacity - capacity/32 keys: a call whose new keys do not ALL fit
// under that limit places none of them (counted in n_full), so that which keys are refused does not
// depend on the order in which the kernels happen to see them.
__host__ __device__ inline int64_t rows_on_offer(uint64_t capacity, int32_t free_n) {
  const int64_t offer = (int64_t)free_n - (int64_t)(capacity >> kReserveShift);
  return offer > 0 ? offer : 0;
}

constexpr uint32_t kAgeEmpty = 0xFFu, kAgeLook = 0u, kAgeModulus = 254u;  // other values of a byte of `oldest`: 1 + unit mod 254
constexpr uint32_t kAgeUnits = 100;
__host__ __device__ inline uint32_t sweep_unit(uint32_t step, uint32_t sweep_q) { return 1u + (step >> sweep_q) % kAgeModulus; }

// A wave of the sweep owns 256 buckets, or 1024 of a large table.
constexpr uint64_t kSweepSmallWave = 256, kSweepLargeWave = 1024, kSweepLargeTable = 1ull << 26;  // buckets, buckets, slots
__host__ __device__ inline uint64_t sweep_wave_buckets(uint64_t capacity) {
  return capacity >= kSweepLargeTable ? kSweepLargeWave : kSweepSmallWave;
}
__host__ __device__ inline uint64_t occupancy_words(uint64_t capacity) { return (capacity + 511) / 512; }

// Large calls on tables whose counters do not age note which counters the missing keys have brought to the threshold, or found
// there: one without the call's mark has not reached it, and the election, which comes after all counts, need not read
// it.  The marks are ordinary stores of bytes: the caches hold the whole array, and the kernel's end brings it together.
// Marks come again every 255 calls, and counters share bytes: a mark only says that the counter is worth a look.  6.8 M
// keys, a million of them kept out: the election 44 -> 36 us.  Where counters age, 690 K keys with two counters each, the
// probe took 2 us longer and the election as long as before.
constexpr uint64_t kReachedMost = 1ull << 20;
__device__ inline uint8_t reached_mark(uint32_t epoch) { return (uint8_t)(1u + epoch % 255u); }

__device__ inline uint64_t shr_or_zero(uint64_t h, uint32_t shift) { return shift >= 64 ? 0 : h >> shift; }

__device__ inline uint64_t bucket_index(const TableView& t, int side, uint64_t key) {
  uint64_t h = mix64(key ^ (side == 0 ? t.s_h0 : t.s_h1));
  return shr_or_zero(h, t.bucket_shift) + (side == 0 ? 0 : t.n_buckets);
}

__device__ inline uint64_t filter_index(const TableView& t, uint64_t key, uint32_t j = 0) {
  return shr_or_zero(mix64(key ^ t.s_filter[j]), t.filter_shift);
}

// Initial value of element j of the row of `key`: uniform on a 2^-27 grid in [-2^-4, 2^-4).
// `base` = mix64(key ^ s_init).  Only exact fp32 operations.
__device__ inline float init_value(uint64_t base, uint32_t j) {
  uint32_t u24 = (uint32_t)(mix64(base + (uint64_t)j) >> 40);
  return ((float)u24 * (1.0f / 8388608.0f) - 1.0f) * 0.0625f;
}

// bfloat16 <-> fp32 on bit patterns; round to nearest even.
__device__ inline uint16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7F800000u) == 0x7F800000u) {
    if (u & 0x007FFFFFu) u |= 0x00400000u;
    return (uint16_t)(u >> 16);
  }
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// agent-scope relaxed atomics on table words (visible across all compute units of the device)
template <typename T>
__device__ inline T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Accesses whose data should not displace others from the 256 MB cache behind the L2s: a pair that nobody
// reads again, results far larger than that cache.
__device__ inline uint2 load_once(const uint2* p) {
  const unsigned long long x = __builtin_nontemporal_load(reinterpret_cast<const unsigned long long*>(p));
  return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
}
__device__ inline void store_float4(float* p, float4 v, bool past_caches) {
  typedef float Vec __attribute__((ext_vector_type(4)));
  if (past_caches)  // the same for the whole launch
    __builtin_nontemporal_store(Vec{v.x, v.y, v.z, v.w}, reinterpret_cast<Vec*>(p));
  else
    *reinterpret_cast<float4*>(p) = v;
}

// LDS words through which the lanes of one wave pass values to each other without a barrier: LDS serves a wave in order,
// only the compiler has to be kept from moving an access or keeping a value (wave_order between what must not swap).
// A volatile pointer does that too, but the accesses are then flat ones, which wait for vector memory as well (sort of
// 690 K pairs, with two of the wave's own LDS words to a round: the training step 175 -> 172 us; 7.6 M IDs 781 -> 768).
template <typename T>
__device__ inline T wave_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename T>
__device__ inline void wave_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ inline void wave_order() {
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  __asm__ volatile("" ::: "memory");
}

__device__ inline unsigned lane_id() { return __lane_id(); }
__device__ inline uint64_t lanes_below() { return (1ull << lane_id()) - 1ull; }

// Inclusive sum over the lanes of a wave, by moves between registers (a shuffle goes through LDS: 130 cycles a step).
// Called by whole waves.
__device__ inline uint32_t wave_sums(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // the lane before, of the row of 16
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // two before
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // last lane of the row before, rows 1 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // last lane of row 1, rows 2 and 3
  return x;
}
// Inclusive maximum, the same way.
__device__ inline uint32_t wave_maxima(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
  return x;
}
// The value of one lane, the same for the whole wave, in all of them.
__device__ inline uint32_t lane_value(uint32_t x, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)lane);
}

// Element w of all sub-lists, one after the other: the list it is in, and how many elements come before that list.  inc: the
// lists' inclusive prefix sums, one per lane; first: the smallest w of the wave (the same for all its lanes).  Called by whole
// waves whose w, of the valid lanes, are neighbours: they are in one list or a few.
__device__ inline uint32_t list_holding(uint32_t inc, uint32_t w, uint32_t first, bool valid, uint32_t* before) {
  uint32_t list = (uint32_t)__popcll(__ballot(inc <= first));  // (no list is left behind the last element)
  *before = list > 0 ? lane_value(inc, list - 1) : 0u;
  uint32_t mine = list;
  for (; list < 64; ++list) {
    const uint32_t end = lane_value(inc, list);
    const bool past = valid && w >= end;
    if (!__ballot(past)) break;
    if (past) {
      mine = list + 1;
      *before = end;
    }
  }
  return mine;
}

// Sum over the lanes of a group of `group` (a power of two, the same for the whole wave), in all of them: moves between
// registers again.  Whole groups call it.  (The partners of a step hold equal sums, so that a mirror image will do for the
// lane whose number differs in one bit; of two copies of a register the swaps leave one with either half's.)
__device__ inline float group_sum(float x, uint32_t group) {
  const auto mate = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  if (group > 1) x += mate(x, std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
  if (group > 2) x += mate(x, std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
  if (group > 4) x += mate(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
  if (group > 8) x += mate(x, std::integral_constant<int, 0x140>{});  // row_mirror
  if (group > 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if (group > 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return x;
}

}  // namespace mono
