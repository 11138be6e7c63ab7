// gather_pool: embedding-row gather with per-bag sum pooling.
//
// A wave owns a few consecutive bags, at most 64.  First every lane loads the bounds and the first
// kIdsInRegs indices of ONE bag (coalesced: the bags of a wave are neighbours in `offsets` and in the
// index array).  Then the wave walks its bags in rounds: a group of lanes takes one bag per round, gets
// the bag's indices from the owner lane by shuffle, reads the rows (one coalesced access of 16 bytes per
// lane and row, kIdsInRegs rows in flight) and writes the pooled row once, in full lines.  Rows wider than
// 64 lanes hold are walked in segments by the whole wave.  A bag longer than kIdsInRegs goes on in steps
// of kIdsInRegs indices, the next step's indices requested before this step's rows are waited for (bags
// of 23 IDs on average, dim 36: 144 us per launch when the rest of a long bag was read one row at a time,
// 20 us so).  A wave whose bags all hold at most two IDs, or one (one-hot slots), issues four or eight rounds of row reads
// together instead (a million bags of one ID, bf16 of dim 64, us: 81 round by round, 67 four together; eight 61 there, and within
// 3 % of four with other tables and dims.  fp32 rows, 4 M uniform ones: of dim 32 52 two by two, 49 one by one, which is what
// eight rounds are if the rows are not held, and 44 together, of dim 64 97, 89 and 83; bags of two, dim 32, 78 two by two and
// 65.  In training steps of a million Zipf IDs of dim 64: 93, 88 and 76, in bags of two 65 and 49).
//
// How many bags a wave owns decides how many waves there are, and the kernel is latency-bound below a few
// thousand of them: 64, where that still leaves kWavesWanted waves (the index loads are then as coalesced as they can be),
// else as few as one round needs (33 K bags of dim 512: one wave per 64 bags was 512 waves on 256 compute units).
// Never more than 4 where a row takes a whole wave, 2 where it takes two pieces of a wave's width, 1 where it takes more: a
// wave of many rounds lasts long, and the chip is idle beside the last ones (249 K bags of one ID, fp32 dim 512, gather and
// update 491 -> 441 us; 293 K bags of four, dim 256, 215 -> 205; 66 K bags of two with 4 and with 1 or 2, dims 512, 768, 1024:
// fp32 78 / 75 us, 117 / 102, 153 / 142, bf16 with 8 / 4 elements a lane 56 / 52, - , 123 / 112).  But twice as many where the
// launch would be a little more than the chip holds (8192 waves, kHeld), up to half as much again: its last
// waves then run alone (33 K bags with 4 and with 8, dim 256, bags of one and four: fp32 13.9 / 13.1, 27.5 / 27.1 us, bf16
// 11.8 / 10.5, 19.7 / 17.7; 36 K of dim 132 10 % each; from 12 K waves on the same).
// Two tables, for the same reason, 32 bags where 8 lanes share a row, 16 where 16 or 32 do (500 K bags of four, dim 32 67 -> 56
// us, dim 64 159 -> 135, dim 128 272 -> 227; smaller dims the same with 64 and 32), and again twice as many where that is a
// little more than the chip holds, of fp32 rows 6144 waves here (130 K bags of eight of dim 64 94 and 82 us, of dim 128 210
// and 193, 250 K of dim 32 94 and 85).
// Large batches are bound by the rows and pooled rows that move behind the L2 (4.7 TB/s at 6.8 M IDs, 5.5 at 26 M, of
// the 6.2 that a plain copy reaches to consecutive addresses).
// Summation is in occurrence order, in fp32.
//
// Where the rows come from is a policy of the kernel:
//   TableRows       int32 row indices into one table (what lookup_or_insert hands out); an index
//                   outside the table counts as absent
//   QuotRemRows     int64 IDs into the two dense tables of the quotient-remainder decomposition
//                   (the paper's hashing baseline, section 3.1): E = E_r[ID mod 2^m] + E_q[ID div 2^m];
//                   an ID outside [0, 2^(2m)) counts as absent
#include "common.h"
#include "kernels.h"

namespace mono {

constexpr int kIdsInRegs = 8;  // (four where two tables' rows are read: see QuotRemRows)
// Positions in a bag, and the IDs of a bag that count.  The walk of a bag steps up to kIdsInRegs past its last ID, and
// a signed step that wrapped there read in front of the caller's IDs (only the two dense tables take calls of so many).
// 64-bit positions would hold more, but their registers cost the two-table kernel a wave in four (329 -> 399 us).
using BagPos = uint32_t;
constexpr BagPos kMostInBag = 0x7FFFFFFFu;
static_assert(kMostInBag + (BagPos)kIdsInRegs > kMostInBag, "the step after the last ID must not wrap");
constexpr uint64_t kWavesWanted = 4096;  // half of what the chip can hold: enough loads in flight to hide their latency

// N consecutive elements of a row as they are stored (one load), and their sum in fp32.
template <typename E, int N>
struct Piece;
template <>
struct Piece<float, 4> {
  float4 v;
  __device__ void clear() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ void hold() {}
  __device__ void add_to(float* a) const {
    a[0] += v.x;
    a[1] += v.y;
    a[2] += v.z;
    a[3] += v.w;
  }
};
// The same, held between the read and the sum: the compiler must not know any more that an absent row is zero.  Where it knows,
// and the sum begins with the row, it adds the row up in the branch that reads it, which waits for it there: reads that were to
// be in flight together wait for one another.  (One value of four elements, which is read into where it stays.)
struct HeldPiece {
  typedef float Bits __attribute__((ext_vector_type(4)));
  Bits v;
  __device__ void clear() { v = Bits(0.f); }
  __device__ void hold() { __asm__ volatile("" : "+v"(v)); }
  __device__ void add_to(float* a) const {
    a[0] += v.x;
    a[1] += v.y;
    a[2] += v.z;
    a[3] += v.w;
  }
};
__device__ inline void add_bf16_pair(uint32_t u, float* a) {
  a[0] += __uint_as_float(u << 16);
  a[1] += __uint_as_float(u & 0xFFFF0000u);
}
template <>
struct Piece<uint16_t, 4> {
  uint2 v;
  __device__ void clear() { v = make_uint2(0u, 0u); }
  __device__ void hold() {}  // (bf16 elements are widened before they are added, outside the branch)
  __device__ void add_to(float* a) const {
    add_bf16_pair(v.x, a);
    add_bf16_pair(v.y, a + 2);
  }
};
template <>
struct Piece<uint16_t, 8> {
  uint4 v;
  __device__ void clear() { v = make_uint4(0u, 0u, 0u, 0u); }
  __device__ void hold() {}
  __device__ void add_to(float* a) const {
    add_bf16_pair(v.x, a);
    add_bf16_pair(v.y, a + 2);
    add_bf16_pair(v.z, a + 4);
    add_bf16_pair(v.w, a + 6);
  }
};

template <typename P, typename E>
__device__ inline void load_piece(P& p, const E* rows, uint64_t row, uint32_t dim, uint32_t col) {
  p.v = *reinterpret_cast<const decltype(p.v)*>(rows + row * dim + col);
}

template <typename E, int N_>
struct TableRows {
  static constexpr int N = N_, kIds = kIdsInRegs;
  static constexpr uint64_t kHeld = 8192;  // waves that run at a time; 0: does not matter
  static constexpr int kSimdWaves = N_ == 4 && sizeof(E) == 4 ? 7 : 1;
  using Id = int32_t;
  const E* rows;
  const int32_t* idx;
  uint32_t cap;
  struct Row {
    std::conditional_t<sizeof(E) == 4, HeldPiece, Piece<E, N>> p;
    __device__ void clear() { p.clear(); }
    __device__ void hold() { p.hold(); }
    __device__ void add_to(float* a) const { p.add_to(a); }
  };
  __device__ Id none() const { return -1; }
  __device__ Id at(int64_t i) const { return idx[i]; }
  __device__ bool present(Id r) const { return (uint32_t)r < cap; }
  __device__ void fetch(Row& x, Id r, uint32_t dim, uint32_t col) const { load_piece(x.p, rows, (uint32_t)r, dim, col); }
};

// kIds_: IDs of a bag whose rows, two each, are asked for in a step of the walk.  Four: with eight their registers leave four
// waves to a SIMD instead of six (bf16: five and eight).  Eight where bags are long, on average, since each step of the walk
// waits for the one before (see kQrBag).  HELD: they are in flight together (see HeldPiece); fp32 rows that are not wait for one
// another, ID by ID, and only the IDs of the next step come beside them (see qr_holds).
template <typename E, int N_, int kIds_, bool HELD = false>
struct QuotRemRows {
  static_assert(!HELD || (sizeof(E) == 4 && N_ == 4), "bf16 rows are in flight together anyway");
  static constexpr int N = N_, kIds = kIds_;
  static constexpr uint64_t kHeld = kIds_ == 4 && sizeof(E) == 4 ? 6144 : 0;
  static constexpr int kSimdWaves = 1;
  using Id = int64_t;
  const E* rem;    // E_r: 2^m rows
  const E* quot;   // E_q: 2^m rows
  const int64_t* ids;
  uint32_t m;
  struct Row {
    std::conditional_t<HELD, HeldPiece, Piece<E, N>> r, q;
    __device__ void clear() {
      r.clear();
      q.clear();
    }
    __device__ void hold() {
      r.hold();
      q.hold();
    }
    __device__ void add_to(float* a) const {  // E_r + E_q first, then the bag's sum
      float e[N];
#pragma unroll
      for (int i = 0; i < N; ++i) e[i] = 0.f;
      r.add_to(e);
      q.add_to(e);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] += e[i];
    }
  };
  __device__ Id none() const { return -1; }
  __device__ Id at(int64_t i) const { return ids[i]; }
  __device__ bool present(Id id) const { return ((uint64_t)id >> (2 * m)) == 0; }
  __device__ void fetch(Row& x, Id id, uint32_t dim, uint32_t col) const {
    load_piece(x.r, rem, (uint64_t)id & ((1ull << m) - 1), dim, col);
    load_piece(x.q, quot, (uint64_t)id >> m, dim, col);
  }
};

template <int N>
__device__ inline void store_pooled(float* out, const float* a, bool past_caches) {
#pragma unroll
  for (int i = 0; i < N; i += 4) store_float4(out + i, make_float4(a[i], a[i + 1], a[i + 2], a[i + 3]), past_caches);
}

// group_log2: log2 of the lanes that share a row; bags_log2: log2 of the bags a wave owns (64 >> group_log2 at
// least); past_caches: how the pooled rows are stored (GatherShape)
template <typename Src>
__global__ __launch_bounds__(256, Src::kSimdWaves) void gather_pool_kernel(Src src, const int64_t* __restrict__ offsets,
                                                          uint64_t n_bags, uint64_t n, uint32_t dim,
                                                          uint32_t group_log2, uint32_t bags_log2,
                                                          bool past_caches, float* __restrict__ out) {
  using Id = typename Src::Id;
  using Row = typename Src::Row;
  constexpr int N = Src::N, kIds = Src::kIds;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t bag_base = wave << bags_log2;
  if (bag_base >= n_bags) return;  // wave-uniform
  const uint32_t lane = lane_id();
  // phase 1: lane <-> bag
  const bool mine = lane < (1u << bags_log2) && bag_base + lane < n_bags;
  // offsets and indices are the caller's: both are bounded (to the n indices, to the table's
  // rows) so that a malformed input gives zeros, not an access out of range
  int64_t s = mine ? offsets[bag_base + lane] : 0;
  int64_t e = mine ? offsets[bag_base + lane + 1] : 0;
  s = s < 0 ? 0 : s;
  e = e > (int64_t)n ? (int64_t)n : e;
  const int len = e > s ? (int)(e - s > (int64_t)kMostInBag ? (int64_t)kMostInBag : e - s) : 0;
  Id id[kIds];
#pragma unroll
  for (int j = 0; j < kIds; ++j) id[j] = j < len ? src.at(s + j) : src.none();
  // phase 2: group <-> bag, one bag per group and round
  const uint32_t group = 1u << group_log2, l = lane & (group - 1u), g = lane >> group_log2;
  const uint32_t bags_per_round = 64u >> group_log2, rounds = (1u << bags_log2) >> (6u - group_log2);
  // Short bags: a round keeps only one or two rows per lane in flight, so as many rounds are issued together as have kIds rows.
  const auto short_bags = [&](auto longest) {
    constexpr int kShort = decltype(longest)::value, kRoundsTogether = kIds / kShort;
    const bool active = l * N < dim;
    for (uint32_t q0 = 0; q0 < rounds; q0 += kRoundsTogether) {
      Row v[kRoundsTogether][kShort];
#pragma unroll
      for (int rr = 0; rr < kRoundsTogether; ++rr) {
        const int from = (int)((q0 + rr) * bags_per_round + g) & 63;
#pragma unroll
        for (int j = 0; j < kShort; ++j) {
          const Id r = __shfl(id[j], from);
          v[rr][j].clear();
          if (q0 + rr < rounds && src.present(r) && active) src.fetch(v[rr][j], r, dim, l * N);
        }
      }
#pragma unroll
      for (int rr = 0; rr < kRoundsTogether; ++rr) {
        float acc[N] = {0.f};
#pragma unroll
        for (int j = 0; j < kShort; ++j) {
          v[rr][j].hold();
          v[rr][j].add_to(acc);
        }
        const uint64_t bag = bag_base + (q0 + rr) * bags_per_round + g;
        if (q0 + rr < rounds && bag < n_bags && active) store_pooled<N>(out + bag * dim + l * N, acc, past_caches);
      }
    }
  };
  if (dim <= 64 * N) {  // (all of this is wave-uniform)
    if (!__ballot(len > 1)) return short_bags(std::integral_constant<int, 1>{});
    if (!__ballot(len > 2)) return short_bags(std::integral_constant<int, 2>{});
  }
  for (uint32_t q = 0; q < rounds; ++q) {
    const int from = (int)(q * bags_per_round + g);
    const BagPos blen = (BagPos)__shfl(len, from);
    const int64_t bs = __shfl(s, from);
    const uint64_t bag = bag_base + (uint32_t)from;
    for (uint32_t col0 = 0; col0 < dim; col0 += 64 * N) {  // one trip unless the row is wider than the wave
      const uint32_t col = col0 + l * N;
      const bool active = col < dim;
      float acc[N] = {0.f};
      Id rid[kIds];
#pragma unroll
      for (int j = 0; j < kIds; ++j) rid[j] = __shfl(id[j], from);
      for (BagPos c = 0;;) {
        Row v[kIds];
#pragma unroll
        for (int j = 0; j < kIds; ++j) {
          v[j].clear();
          if (src.present(rid[j]) && active) src.fetch(v[j], rid[j], dim, col);
        }
        c += kIds;
        const bool more = c < blen;
        if (more) {  // a long bag: its next indices, straight from memory (the group's lanes ask for the same words)
#pragma unroll
          for (int j = 0; j < kIds; ++j) rid[j] = c + j < blen ? src.at(bs + c + j) : src.none();
        }
#pragma unroll
        for (int j = 0; j < kIds; ++j) {
          v[j].hold();
          v[j].add_to(acc);
        }
        if (!more) break;
      }
      if (bag < n_bags && active) store_pooled<N>(out + bag * dim + col, acc, past_caches);
    }
  }
}

// Lanes per row, bags per wave, the grid of a launch, and whether the pooled rows go past the caches.  The layer that
// takes them reads them next, so what counts is the gather and that layer together, with caches that the rest of a step
// has filled with something else.  Rows of four elements per lane go past them beyond kPooledCached bytes, three
// quarters of the cache behind the L2s; the layer would then find little of them there (gather and a layer that reads
// all of it, through the caches and past them: 100 MB of dim 32 117 and 126 us, 128 MB 142 and 150, 192 MB 204 and 198,
// 400 MB 367 and 363; dim 256 192 MB 200 and 207, 256 MB 257 and 259; bf16 of dim 64 100 MB 96 and 110, 192 MB 177 and
// 179, 240 MB 214 and 210, 400 MB 341 and 321).  Rows of eight elements per lane never do: a lane stores them in two
// pieces, which past the caches reach the memory as half lines (bf16 of dim 512, 66 MB 71 and 91 us, 400 MB 350 and 429).
constexpr uint64_t kPooledCached = 192ull << 20;
constexpr uint64_t kMostWaves = (1ull << 26) - 4;  // a launch has fewer than 2^32 threads, in whole blocks of four waves
struct GatherShape {
  uint32_t group_log2 = 0, bags_log2 = 6;
  bool past_caches;
  uint64_t waves;
  GatherShape(uint32_t dim, uint32_t n_per_lane, uint64_t n_bags, uint32_t ids = kIdsInRegs, uint64_t held = 0)
      : past_caches(n_per_lane == 4 && n_bags * dim * sizeof(float) > kPooledCached) {
    while (group_log2 < 6 && (n_per_lane << group_log2) < dim) ++group_log2;
    const uint32_t pieces = (dim + 64 * n_per_lane - 1) / (64 * n_per_lane);
    if (group_log2 == 6)
      bags_log2 = pieces == 1 ? 2 : (pieces == 2 ? 1 : 0);
    else if (group_log2 >= 3 && ids < (uint32_t)kIdsInRegs)
      bags_log2 = group_log2 == 3 ? 5 : 4;
    while (bags_log2 > 6 - group_log2 && (n_bags >> bags_log2) < kWavesWanted) --bags_log2;
    const auto waves_of = [&](uint32_t lg) { return (n_bags + (1ull << lg) - 1) >> lg; };
    if (bags_log2 < 6 && held != 0 && waves_of(bags_log2) >= held && waves_of(bags_log2) <= held + held / 2) ++bags_log2;
    while (bags_log2 < 6 && waves_of(bags_log2) > kMostWaves) ++bags_log2;
    waves = waves_of(bags_log2);
  }
};

template <typename Src>
static hipError_t queue_gather(const Src& src, const int64_t* d_offsets, uint64_t n_bags, uint64_t n, uint32_t dim,
                               float* d_out, hipStream_t stream, Profiler* prof) {
  const GatherShape sh(dim, Src::N, n_bags, Src::kIds, Src::kHeld);
  MONO_LAUNCH(prof, K_GATHER_POOL, stream, gather_pool_kernel<Src>, dim3((unsigned)((sh.waves + 3) / 4)), dim3(256), src,
              d_offsets, n_bags, n, dim, sh.group_log2, sh.bags_log2, sh.past_caches, d_out);
  return hipGetLastError();
}

// bf16 rows wider than 256 elements are read eight elements per lane (dim 512: one
// access of the wave per row instead of two, 35.6 -> 31.8 us for 33 K bags), others four (dim 64, one ID per
// bag: 64 us with four, 76 with eight, whose registers leave fewer waves)
hipError_t launch_gather_pool(const TableView& t, const int32_t* d_rows, uint64_t n, const int64_t* d_offsets,
                              uint64_t n_bags, float* d_out, hipStream_t stream, Profiler* prof) {
  if (n_bags == 0) return hipSuccess;
  const uint32_t cap = (uint32_t)t.capacity;
  if (!t.bf16)
    return queue_gather(TableRows<float, 4>{(const float*)t.rows, d_rows, cap}, d_offsets, n_bags, n, t.dim, d_out, stream,
                        prof);
  const uint16_t* rows = (const uint16_t*)t.rows;
  if (t.dim >= 512)
    return queue_gather(TableRows<uint16_t, 8>{rows, d_rows, cap}, d_offsets, n_bags, n, t.dim, d_out, stream, prof);
  return queue_gather(TableRows<uint16_t, 4>{rows, d_rows, cap}, d_offsets, n_bags, n, t.dim, d_out, stream, prof);
}

// Average bags from which on eight IDs' rows are in flight.  With eight and with four: 6.8 M Zipf IDs in bags of four,
// dim 32, 327 and 278 us; 0.4 to 8 M IDs in bags of two to five, dims 64 to 512, 15 to 50 % longer with eight; bags of 16
// and 30, uniform IDs, dims 16 and 64, 150 and 159, 62 and 63, 141 and 145; 3037 bags of 28, dim 128, 19.6 and 20.5.  bf16
// rows of up to 32 elements are short of neither registers nor waves: bags of five, dim 16 376 and 390, of two, dim 32, 45 and 38.
// Shorter bags of fp32 rows that share a wave with three others or more, where there are so many that the chip is full twice
// over: bags of eight, uniform IDs, 500 K of dim 32 164 and 171, 250 K of dim 64 153 and 160 (90 K of dim 128 142 and 134, 66 K
// of dim 64 57 and 45).
// And of rows of more than two pieces of a wave's width, which a wave takes bag by bag: bags of eight, eight and four: bf16 of dim
// 1024, 1000 bags 9.0 and 10.0 us, 32 K 159 and 165, fp32 16.9 and 17.5, 430 and 445, at worst (2 to 4 K bags) 3 % the other way.  Bags
// of nine to eleven, two steps of eight or three of four, there too only where there are many: 100 bags 13.6 and 12.9 us.
// Of two pieces only fp32 rows of such many waves (dim 512, 64 K bags 301 and 311 us, 12 K 65 and 61).
constexpr uint64_t kQrBag = 12, kQrBagNarrow = 3, kQrBagMany = 6;
inline bool qr_takes_eight(uint64_t n, uint64_t n_bags, uint32_t dim, bool bf16) {
  const GatherShape four(dim, 4, n_bags, 4);
  const bool many = four.waves >= 2 * QuotRemRows<float, 4, 4>::kHeld;
  uint64_t bag = kQrBag;
  if (dim > 2 * 64 * 4) {
    if (many || n <= kIdsInRegs * n_bags) bag = kQrBagMany;
  } else if (bf16) {
    if (dim <= 32) bag = kQrBagNarrow;
  } else if (many && (four.group_log2 <= 4 || dim > 64 * 4)) {
    bag = kQrBagMany;
  }
  return n / n_bags >= bag;
}

// fp32 rows that eight lanes or more share are held where the chip is full twice over.  Bags of one, of zero to three, of four,
// Poisson(5), and of one but for every 512th, which holds 200; not held and held, us.  1.6 M of dim 32: uniform IDs 95 / 92, 126 /
// 121, 268 / 271, 340 / 338, 452 / 297, Zipf 70 / 69, 89 / 87, 176 / 173, 250 / 217, 379 / 260.  197 K of dim 128: 55 / 48, 78 / 73,
// 169 / 153, 207 / 191, 190 / 140 and 42 / 39, 62 / 55, 109 / 95, 138 / 117, 160 / 116.  98 K of dim 512: 94 / 93, 113 / 111,
// 255 / 256, 313 / 314, 609 / 455 and 73 / 73, 97 / 91, 182 / 172, 223 / 214, 488 / 370.  6.8 M IDs in bags of four, dim 32, Zipf,
// 217 / 206.  The most that is lost is 3 %, of uniform IDs (197 K bags of two, dim 256, 141 / 146).  (Two IDs a step, not held, let
// eight waves share a SIMD: 6 % less than four for Poisson bags of Zipf IDs, but 5 to 8 % more for the few long ones.)
// Elsewhere rows are not held: fewer waves take up to 5 % longer so where rows are wide and IDs uniform (6 K bags of five, dim
// 1024, 42.7 / 43.0, Zipf 30.4 / 32.0), and rows of fewer lanes up to 2 %; long bags of few waves would gain (3333 of 30, dim 32,
// 15.0 / 9.4).
inline bool qr_holds(uint64_t n_bags, uint32_t dim) {
  const GatherShape four(dim, 4, n_bags, 4);
  return four.group_log2 >= 3 && four.waves >= 2 * QuotRemRows<float, 4, 4>::kHeld;
}

hipError_t launch_qr_gather_pool(const void* d_rem, const void* d_quot, uint32_t log2_rows, uint32_t dim, bool bf16,
                                 const int64_t* d_ids, uint64_t n, const int64_t* d_offsets, uint64_t n_bags,
                                 float* d_out, hipStream_t stream) {
  if (n_bags == 0) return hipSuccess;
  const bool eight = qr_takes_eight(n, n_bags, dim, bf16);
  const auto queue = [&](const auto& src) { return queue_gather(src, d_offsets, n_bags, n, dim, d_out, stream, nullptr); };
  if (!bf16) {
    const float *rem = (const float*)d_rem, *quot = (const float*)d_quot;
    if (eight) return queue(QuotRemRows<float, 4, kIdsInRegs>{rem, quot, d_ids, log2_rows});
    return qr_holds(n_bags, dim) ? queue(QuotRemRows<float, 4, 4, true>{rem, quot, d_ids, log2_rows})
                                 : queue(QuotRemRows<float, 4, 4>{rem, quot, d_ids, log2_rows});
  }
  const uint16_t *rem = (const uint16_t*)d_rem, *quot = (const uint16_t*)d_quot;
  return eight ? queue(QuotRemRows<uint16_t, 4, kIdsInRegs>{rem, quot, d_ids, log2_rows})
               : queue(QuotRemRows<uint16_t, 4, 4>{rem, quot, d_ids, log2_rows});
}

}  // namespace mono
