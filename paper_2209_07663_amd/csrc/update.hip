// apply_grad_adagrad: duplicate-ID gradient scatter-reduce + row-wise Adagrad.
//
//   sort         grouping of (row, bag) by row, stable: the occurrences of a row become one run (the
//                pooled gradient of bag b is the gradient of each of its occurrences; the first pass
//                finds the bag of every occurrence from the offsets); dropped occurrences (row -1) are
//                left out
//   order_tiles  (many gradients, each of several occurrences) the order in which seg_reduce takes its tiles
//   seg_reduce   the sorted sequence is cut into tiles, a block each, and a tile into chunks, one for each lane
//                group of the block (dim/4 lanes, four elements each); the group loads its chunk's pairs at once, then walks
//                them with four or eight gradient rows in flight, summing grad[bag] along each run.  A run that lies
//                inside the chunk is complete: Adagrad is applied at once.  A run that crosses a
//                chunk border leaves a partial sum; a segmented scan over the block's chunks then joins the
//                partials of runs that stay inside the block's tile (Adagrad again) and only runs
//                that cross a BLOCK border leave partials in global memory (at most two per block)
//   combine      one block per run that crosses block borders: adds its partials (lane groups in
//                parallel, then across groups) and applies Adagrad
// A hot ID with 10^5..10^6 occurrences is thus reduced as chunk sums -> tile sums -> total, never
// serially, and everything is deterministic: no floating-point atomics.
// The store that writes a row's new accumulator also carries the number of the current
// synchronisation window: that is the row's "touched" mark (paper section 2.2.3), at no extra cost.
//
// Partial slots of tile u in global memory: slot A = 2u ("run that started before this tile and ends inside it") and slot
// B = 2u + 1 ("run that continues past the end of this tile"; flag kHeadFlag if it also starts inside it).
#include "common.h"
#include "kernels.h"
#include "table_ops.h"

namespace mono {

constexpr uint32_t kHeadFlag = 0x80000000u;
constexpr uint32_t kReduceWaves = 4;  // waves of a block of seg_reduce
constexpr uint64_t kReduceFew = 1024; // (see seg_reduce_kernel)

// seg_reduce reads and writes embedding rows past the caches where the batch's occurrences come to more bytes of
// rows than the 256 MB cache behind the L2s holds: each row is used once and would not be there for the next
// lookup, and the gradients, which several occurrences share, stay there instead (26 M pairs of dim 64: 1790 ->
// 1700 us; 6.8 M of dim 32: 250 -> 244 and what runs after it a little faster; with nothing in the caches but the gradients
// that a layer has just written, 270 MB to 1.6 GB of rows of dims 32, 128 and 512 and of bf16 rows of dim 64: 2 to 8 %).
constexpr uint64_t kRowsCached = 256ull << 20;

// Four elements of a row: their bits (one access), and the same as floats.  PAST: past the caches (see kRowsCached).
template <typename E>
struct Quad;
template <>
struct Quad<float> {
  typedef float Bits __attribute__((ext_vector_type(4)));
  __device__ static inline float4 open(Bits u) { return make_float4(u.x, u.y, u.z, u.w); }
  __device__ static inline Bits pack(float4 v) { return Bits{v.x, v.y, v.z, v.w}; }
};
template <>
struct Quad<uint16_t> {
  typedef uint32_t Bits __attribute__((ext_vector_type(2)));
  __device__ static inline float4 open(Bits u) {
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xFFFF0000u));
  }
  __device__ static inline Bits pack(float4 v) {
    return Bits{(uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16),
                (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16)};
  }
};
template <typename E, bool PAST>
__device__ inline float4 load_row4(const E* rows, uint32_t row, uint32_t dim, uint32_t l) {
  const auto* p = reinterpret_cast<const typename Quad<E>::Bits*>(rows + (uint64_t)row * dim + l * 4);
  return Quad<E>::open(PAST ? __builtin_nontemporal_load(p) : *p);
}
template <typename E, bool PAST>
__device__ inline void store_row4(E* rows, uint32_t row, uint32_t dim, uint32_t l, float4 v) {
  auto* p = reinterpret_cast<typename Quad<E>::Bits*>(rows + (uint64_t)row * dim + l * 4);
  if constexpr (PAST)
    __builtin_nontemporal_store(Quad<E>::pack(v), p);
  else
    *p = Quad<E>::pack(v);
}

// lr / (sqrt(acc) + eps) with the hardware square root and reciprocal (1 ulp each: the update is
// compared at 1e-5, and this runs once per distinct row inside the serial walk of seg_reduce)
__device__ inline float step_scale(float acc, float lr, float eps) {
  return lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(acc) + eps);
}

// A lane's share of a row: SEG pieces of four elements, piece q at elements (q * 64 + l) * 4.  Rows of
// at most 256 elements have one piece per lane (SEG = 1, lane groups of up to 64 lanes); wider rows
// (512, 768, 1024 elements) are held by the whole wave with SEG = 2, 3, 4.
template <int SEG>
struct RowVec {
  float4 v[SEG];
  __device__ inline void zero() {
#pragma unroll
    for (int q = 0; q < SEG; ++q) v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __device__ inline void add(const RowVec& o) {
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      v[q].x += o.v[q].x;
      v[q].y += o.v[q].y;
      v[q].z += o.v[q].z;
      v[q].w += o.v[q].w;
    }
  }
  __device__ inline void add_xor(uint32_t lanes) {  // the share of the lane whose number differs by `lanes` (xor)
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      v[q].x += __shfl_xor(v[q].x, (int)lanes);
      v[q].y += __shfl_xor(v[q].y, (int)lanes);
      v[q].z += __shfl_xor(v[q].z, (int)lanes);
      v[q].w += __shfl_xor(v[q].w, (int)lanes);
    }
  }
  __device__ inline RowVec from_up(uint32_t lanes) const {  // the share of the lane `lanes` before this one
    RowVec o;
#pragma unroll
    for (int q = 0; q < SEG; ++q)
      o.v[q] = make_float4(__shfl_up(v[q].x, lanes), __shfl_up(v[q].y, lanes), __shfl_up(v[q].z, lanes), __shfl_up(v[q].w, lanes));
    return o;
  }
  __device__ inline float sum_sq() const {
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < SEG; ++q) ss += v[q].x * v[q].x + v[q].y * v[q].y + v[q].z * v[q].z + v[q].w * v[q].w;
    return ss;
  }
};

// piece q of a vector of dim4 float4 (dim4 = dim / 4) held by lane l; `p` points at the vector
template <int SEG>
__device__ inline RowVec<SEG> load_vec(const float4* p, uint32_t l, bool active) {
  RowVec<SEG> r;
#pragma unroll
  for (int q = 0; q < SEG; ++q) r.v[q] = active ? p[q * 64 + l] : make_float4(0.f, 0.f, 0.f, 0.f);
  return r;
}
template <int SEG>
__device__ inline void store_vec(float4* p, uint32_t l, bool active, const RowVec<SEG>& r) {
#pragma unroll
  for (int q = 0; q < SEG; ++q)
    if (active) p[q * 64 + l] = r.v[q];
}
template <typename E, int SEG, bool PAST>
__device__ inline RowVec<SEG> load_row(const E* rows, uint32_t row, uint32_t dim, uint32_t l, bool active) {
  RowVec<SEG> r;
#pragma unroll
  for (int q = 0; q < SEG; ++q)
    r.v[q] = active ? load_row4<E, PAST>(rows, row, dim, q * 64 + l) : make_float4(0.f, 0.f, 0.f, 0.f);
  return r;
}

// w -= scale * g on the lane's share of row `row`
template <typename E, int SEG, bool PAST>
__device__ inline void update_row(E* rows, uint32_t row, uint32_t dim, uint32_t l, const RowVec<SEG>& w,
                                  const RowVec<SEG>& g, float scale) {
#pragma unroll
  for (int q = 0; q < SEG; ++q) {
    float4 nw = w.v[q];
    nw.x = fmaf(-scale, g.v[q].x, nw.x);
    nw.y = fmaf(-scale, g.v[q].y, nw.y);
    nw.z = fmaf(-scale, g.v[q].z, nw.z);
    nw.w = fmaf(-scale, g.v[q].w, nw.w);
    store_row4<E, PAST>(rows, row, dim, q * 64 + l, nw);
  }
}

// Row-wise Adagrad on one row by one lane group; g = this lane's share of the gradient (zero in
// lanes beyond dim), w and acc what the row and its accumulator hold.  acc += mean_j g_j^2; w_j -= lr * g_j / (sqrt(acc) + eps).
template <typename E, int SEG, bool PAST>
__device__ inline void adagrad_row(const TableView& t, uint32_t row, const RowVec<SEG>& w, float acc, const RowVec<SEG>& g,
                                   bool active, uint32_t l, uint32_t group, float lr, float eps) {
  const float ss = group_sum(g.sum_sq(), group);
  acc += ss / (float)t.dim;
  if (active) update_row<E, SEG, PAST>(reinterpret_cast<E*>(t.rows), row, t.dim, l, w, g, step_scale(acc, lr, eps));
  if (l == 0) t.state[row] = RowState{acc, t.sync_epoch};  // trained in this window
}

// Order in which seg_reduce takes its tiles where the gradients are more than the caches hold and each is the gradient of
// several occurrences: first the tiles that hold several rows, which read gradients from anywhere, then those of one hot row,
// by the bag that they begin with.  (A row's pairs are in the order of the bags, so that tiles of different hot rows that run
// together read the same part of the gradients.)  Of the latter an XCD takes an eighth of the bags, in order: neighbouring
// blocks run on different XCDs, which do not share an L2.  26 M pairs of dim 64, Zipf 1.1, half of them in such tiles, 1.3 GB
// of gradients: seg_reduce 1690 us without, 1540 without the eighths, 1530 so; with the tiles of several rows last 1550; tiles
// of 512 pairs 1520, but 30 us more to combine.
// All blocks look for the tiles' bins (bags, in equal parts), and the one that finishes last counts and orders them: the
// looking is what takes memory's time, and 26 K tiles are 25 for each of a block's threads (19 us in all).  Where fewer than
// one tile in 16 is of one row the order stays as it is.
constexpr uint32_t kOrderThreads = 1024, kOrderBins = 2 * kOrderThreads;  // (bin 0: several rows, or not full)

__global__ __launch_bounds__(kOrderThreads) void order_tiles_kernel(Control* __restrict__ ctl, const uint2* __restrict__ pair_a,
                                                                    const uint2* __restrict__ pair_b, uint32_t tiles,
                                                                    uint32_t tile, uint64_t n_bags, uint32_t launched,
                                                                    uint32_t max_bits, uint32_t* bins, uint32_t* __restrict__ order) {
  __shared__ uint32_t s_at[kOrderBins], s_wave[kOrderThreads / 64], s_several[kOrderThreads / 64], s_hot, s_last;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
  const SortPlan plan = make_sort_plan(ctl->hwm, max_bits ? max_bits : 32);
  if (plan.passes > launched) return;  // (nothing is sorted; see seg_reduce_kernel)
  const uint2* __restrict__ sp = max_bits == 0 || plan.passes % 2 ? pair_b : pair_a;
  const uint64_t n = ctl->scratch[kValidPairs], t0 = ((uint64_t)blockIdx.x * kOrderThreads + tid) * tile;
  const uint32_t mine = blockIdx.x * kOrderThreads + tid;
  if (tid == 0) s_hot = 0;
  for (uint32_t b = tid; b < kOrderBins; b += kOrderThreads) s_at[b] = 0;
  uint32_t bin = 0;
  if (mine < tiles && t0 + tile <= n) {
    const uint2 first = sp[t0];
    if (first.x == sp[t0 + tile - 1].x) bin = 1u + (uint32_t)((uint64_t)first.y * (kOrderBins - 1) / n_bags);
  }
  if (mine < tiles) st_agent(&bins[mine], bin);
  wait_all_memory_ops();
  __syncthreads();
  const uint64_t of_wave = __ballot(bin != 0);
  if (lane == 0 && of_wave) atomicAdd(&s_hot, (uint32_t)__popcll(of_wave));
  __syncthreads();
  if (tid == 0) {  // low half: blocks; high half: tiles of one row
    const unsigned long long one = (unsigned long long)s_hot << 32 | 1ull, sum = atomicAdd(&ctl->scratch[kOrderDone], one) + one;
    s_last = (uint32_t)sum == gridDim.x;
    s_hot = (uint32_t)(sum >> 32);
  }
  __syncthreads();
  if (!s_last) return;
  const bool ordered = s_hot > tiles / 16;
  if (tid == 0) {
    ctl->scratch[kOrderDone] = 0;
    if (!ordered) ctl->scratch[kOrdered] = 0;
  }
  if (!ordered) return;
  constexpr uint32_t kAhead = 32;  // tiles of a thread whose bins it holds: all of a batch of 32 M pairs
  uint32_t held[kAhead], several = 0;  // tiles of bin 0, of this wave: they are many, and need no word that all add to
  for (uint32_t pass = 0; pass < 2; ++pass) {
    for (uint32_t u0 = 0; u0 < tiles; u0 += kAhead * kOrderThreads) {
      if (pass == 0 || tiles > kAhead * kOrderThreads) {
#pragma unroll
        for (uint32_t q = 0; q < kAhead; ++q) {
          const uint32_t u = u0 + q * kOrderThreads + tid;
          held[q] = u < tiles ? ld_agent(&bins[u]) : kOrderBins;
        }
      }
#pragma unroll
      for (uint32_t q = 0; q < kAhead; ++q) {
        if (u0 + q * kOrderThreads >= tiles) break;  // block-uniform
        const uint64_t none = __ballot(held[q] == 0);
        uint32_t at = several + (uint32_t)__popcll(none & lanes_below());
        several += (uint32_t)__popcll(none);
        if (held[q] - 1u < kOrderBins - 1u) at = atomicAdd(&s_at[held[q]], 1u);
        if (pass == 1 && held[q] < kOrderBins) order[at] = u0 + q * kOrderThreads + tid;
      }
    }
    if (pass == 1) break;
    if (lane == 0) s_several[wave] = several;
    __syncthreads();
    uint32_t first = 0, all = 0;
    for (uint32_t w = 0; w < kOrderThreads / 64; ++w) {
      if (w == wave) first = all;
      all += s_several[w];
    }
    several = first;
    const uint32_t c0 = s_at[2 * tid], c1 = s_at[2 * tid + 1], x = wave_sums(c0 + c1);
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    uint32_t at = all + x - c0 - c1;
    for (uint32_t w = 0; w < wave; ++w) at += s_wave[w];
    s_at[2 * tid] = at;
    s_at[2 * tid + 1] = at + c0;
    if (tid == 0) ctl->scratch[kOrdered] = all + 1ull;
    __syncthreads();
  }
}

// The tile of a block: an XCD's blocks take an eighth of the tiles of one row.
__device__ inline uint32_t tile_of_block(const uint32_t* __restrict__ order, uint64_t ordered, uint32_t block, uint32_t tiles) {
  if (!order || ordered == 0) return block;
  const uint32_t several = (uint32_t)(ordered - 1), share = (tiles - several) / 8, x = block - several;
  return order[block >= several && x < 8 * share ? several + x % 8 * share + x / 8 : block];
}

// A small batch is bound by the chain of what waits for what: the pairs are asked for beside the words that tell how many there
// are, and the squares of a row are summed by moves between registers (by shuffles through LDS, 130 cycles a step, eight rows
// of dim 32 held a lane group for two microseconds).  26 K pairs of dim 32 10.3 -> 8.5 us, 204 K of dim 16 13.6 -> 11.9, 690 K
// of dim 36 29.4 -> 27.4.
// GLOG = log2(lanes per row), SEG = pieces of four elements per lane (1 unless GLOG == 6).  A block of 256
// threads owns a tile of `tile` consecutive sorted pairs, a group an equal chunk of it; the host picks the size
// of the tile so that small batches still fill the machine.
// FEW: there are no more tiles than kReduceFew, which all run at a time with either number of waves a SIMD, so that a chunk's
// pairs are all asked for together (26 K pairs of dim 32 8.6 and 9.2 us, 1600 of bf16 dim 48 1.2 less).
template <typename E, int GLOG, int SEG, bool PAST, bool FEW>
__global__ __launch_bounds__(256) void seg_reduce_kernel(TableView t, const uint2* __restrict__ pair_a,
                                                         const uint2* __restrict__ pair_b, uint64_t n,
                                                         const float* __restrict__ grad, float lr, float eps,
                                                         float* __restrict__ part, uint32_t* __restrict__ part_row,
                                                         uint32_t tile, uint32_t launched, uint32_t max_bits,
                                                         const uint32_t* __restrict__ order) {
  static_assert(SEG == 1 || GLOG == 6, "rows wider than 256 elements are held by a whole wave");
  extern __shared__ float4 s_mem[];  // [groups_per_block + waves][dim / 4] vectors, the tile's pairs
  using Vec = RowVec<SEG>;
  constexpr uint32_t group = 1u << GLOG, gpb = 256u >> GLOG;  // groups (= chunks) per block
  const uint32_t chunk = tile >> (8 - GLOG);
  // Gradient rows in flight per lane, each with the embedding row it may end in.  Eight where rows go past the caches, which is
  // bound by memory; else four, which leave registers for seven waves a SIMD instead of four: such a kernel waits and computes
  // in turn (with eight and with four, us: 500 K pairs of bf16 dim 128 54 and 43, 945 K of dim 64 82 and 72, 755 K of dim 36 91
  // and 84; past the caches 6.8 M of fp32 dim 32 188 and 193, 26 M of dim 64 1500 and 1527).  Rows in pieces: four, bf16 two
  // (update of 400 K pairs with two and with four, of dim 512, 768, 1024: fp32 309 / 307, 474 / 466, 628 / 610 us, with hot rows
  // 267 / 260, 382 / 365, 498 / 476; bf16 255 / 314, 387 / 473, 535 / 738.  Batches of up to 98 K pairs the same way or
  // within 2 us)
  constexpr int kMany = PAST || FEW ? 8 : 4;
  constexpr int kBatch = SEG > 1 ? (sizeof(E) == 2 ? 2 : 4) : ((int)group < kMany ? (int)group : kMany);
  // Gradient rows in flight where no run ends among them, and no embedding row is wanted: what hot rows are, mostly (690 K
  // pairs of dim 36, many of them of hot rows: 23.3 -> 20.4 us; 26 M of dim 64 1524 -> 1500).  Not for rows in pieces (98 K
  // pairs of bf16 dim 512 48 -> 50), nor of up to 16 elements, whose chunks are short (204 K of dim 16 11.9 -> 12.8).
  constexpr int kLong = SEG > 1 || group < 8 || FEW ? 0 : 8;
  // The tile's sorted pairs, and the rows of the pairs before and after it.  Where neither the place of the sort's result nor the
  // order of the tiles is the device's to say they are asked for beside the words that tell how many pairs remain: what lies
  // behind those is read, and left out below.
  const bool told = max_bits == 0 && !order;
  uint2 ahead[kReduceTile / 256];
  uint32_t edge = kNoRow;
  const auto ask = [&](const uint2* __restrict__ from, uint64_t first) {
    if (threadIdx.x < 2) {
      const uint64_t at = threadIdx.x == 0 ? first - 1 : first + tile;  // (first - 1 of the first tile is beyond every n)
      if (at < n) edge = from[at].x;
    }
#pragma unroll
    for (uint32_t m = 0; m < kReduceTile / 256; ++m) {
      const uint32_t j = m * 256u + threadIdx.x;
      if (j < tile && first + j < n) ahead[m] = from[first + j];
    }
  };
  if (told) ask(pair_b, (uint64_t)blockIdx.x * tile);
  const SortPlan plan = make_sort_plan(t.ctl->hwm, max_bits ? max_bits : 32);  // (max_bits == 0: no radix passes)
  if (plan.passes > launched) {  // the host's bound on the high-water mark was too low: nothing is sorted, nothing is touched
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&t.ctl->n_lost, 1ull);
    if (threadIdx.x == 0) {
      part_row[2 * (uint64_t)blockIdx.x] = kNoRow;
      part_row[2 * (uint64_t)blockIdx.x + 1] = kNoRow;
    }
    return;
  }
  const uint32_t at_tile = tile_of_block(order, t.ctl->scratch[kOrdered], blockIdx.x, gridDim.x);
  const uint32_t hwm = plan.hwm;
  n = t.ctl->scratch[kValidPairs];  // the sort left the dropped occurrences out
  const uint32_t g = threadIdx.x >> GLOG, l = threadIdx.x & (group - 1u);
  const uint32_t dim4 = t.dim >> 2;
  float4* s_vec = s_mem;                   // a group's partial of the run that ends in its chunk
  float4* s_carry = s_mem + gpb * dim4;    // a wave's sum over the run that continues past its last chunk
  const uint64_t n_chunks = (n + chunk - 1) / chunk;
  const uint64_t c0 = (uint64_t)at_tile * gpb;  // first chunk of this block's tile
  const uint64_t c = c0 + g;
  const uint32_t chunks_here = (uint32_t)(n_chunks - c0 < gpb ? n_chunks - c0 : gpb);
  const bool active = l < dim4;
  const float4* g4 = reinterpret_cast<const float4*>(grad);

  // ---- phase 0: the tile's sorted pairs -> LDS (coalesced) ---------------------------------------
  uint2* s_pairs = reinterpret_cast<uint2*>(s_carry + kReduceWaves * dim4);
  __shared__ uint32_t s_edge[2];
  {
    const uint64_t t0 = (uint64_t)at_tile * tile;
    if (!told) ask(max_bits == 0 || plan.passes % 2 ? pair_b : pair_a, t0);  // (where the sort left its result)
    if (threadIdx.x < 2) s_edge[threadIdx.x] = (threadIdx.x == 0 ? t0 - 1 : t0 + tile) < n ? edge : kNoRow;
#pragma unroll
    for (uint32_t m = 0; m < kReduceTile / 256; ++m) {
      const uint32_t j = m * 256u + threadIdx.x;
      if (j < tile) s_pairs[j] = t0 + j < n ? ahead[m] : make_uint2(kNoRow, 0u);
    }
  }
  __syncthreads();

  // ---- phase 1: every group reduces the runs of its chunk -------------------------------------
  uint32_t a_row = kNoRow;      // the run that started before this chunk and ends in it
  uint32_t b_row = kNoRow;      // the run that continues past the end of this chunk,
  bool b_head = false;          // and does it start in this chunk?
  Vec sum;
  sum.zero();
  if (c < n_chunks) {
    const uint64_t cs = c * chunk;
    const uint32_t count = (uint32_t)(n - cs < chunk ? n - cs : chunk);
    const uint2* mine = s_pairs + g * chunk;  // this group's chunk
    const uint32_t before = g == 0 ? s_edge[0] : mine[-1].x;
    const uint32_t after = g == gpb - 1 ? s_edge[1] : mine[chunk].x;  // (kNoRow past the last pair)
    const uint32_t first = mine[0].x;
    const bool first_head_in = cs == 0 || before != first;
    uint32_t run = first;
    bool head_in = first_head_in;
    E* rows = reinterpret_cast<E*>(t.rows);
    const float inv_dim = 1.0f / (float)t.dim;
    for (uint32_t p0 = 0; p0 < count;) {  // position of the batch in the chunk
      // nothing ends in the next kLong pairs of any group of the wave (a row's pairs are neighbours): only gradients are
      // read
      const uint32_t row = mine[p0].x;
      if (kLong > 0 && !__ballot(p0 + kLong > count || row != (p0 + kLong < count ? mine[p0 + kLong].x : after))) {
        Vec v[kLong > 0 ? kLong : 1];
#pragma unroll
        for (int u = 0; u < kLong; ++u)
          v[u] = load_vec<SEG>(g4 + (uint64_t)mine[p0 + u].y * dim4, l, row < hwm && active);
        if (row != run) {
          run = row;
          head_in = true;
          sum.zero();
        }
#pragma unroll
        for (int u = 0; u < kLong; ++u) sum.add(v[u]);
        p0 += kLong;
        continue;
      }
      uint32_t kx[kBatch + 1], ky[kBatch];
      Vec v[kBatch], w[kBatch];
      float a[kBatch];
      bool tail[kBatch], apply[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const uint2 kv = p0 + (uint32_t)u < chunk ? mine[p0 + u] : make_uint2(kNoRow, 0u);
        kx[u] = kv.x;
        ky[u] = kv.y;
      }
      kx[kBatch] = p0 + kBatch < count ? mine[p0 + kBatch].x : after;
      // everything the batch needs from memory is requested before anything is consumed: the
      // gradient row of every pair and, for every run that ends in the batch and lies inside the
      // chunk, its embedding row and accumulator.  (bf16 rows are widened in the branch that reads them, which
      // waits for them there: where several runs end, their reads follow one another.)
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const bool in = p0 + (uint32_t)u < count;
        const uint32_t next = p0 + (uint32_t)u + 1 < count ? kx[u + 1] : after;
        tail[u] = in && next != kx[u];
        apply[u] = tail[u] && kx[u] < hwm && (kx[u] != first || first_head_in);
        v[u] = load_vec<SEG>(g4 + (uint64_t)ky[u] * dim4, l, in && kx[u] < hwm && active);
        w[u] = load_row<E, SEG, PAST>(rows, kx[u], t.dim, l, apply[u] && active);
        a[u] = apply[u] ? t.state[kx[u]].acc : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (p0 + (uint32_t)u < count) {
          if (kx[u] != run) {
            run = kx[u];
            head_in = true;
            sum.zero();
          }
          sum.add(v[u]);
          if (tail[u]) {
            if (apply[u]) {  // the run lies inside the chunk: row-wise Adagrad at once
              const float ss = group_sum(sum.sum_sq(), group);
              const float acc = a[u] + ss * inv_dim;
              const float scale = step_scale(acc, lr, eps);
              if (active) update_row<E, SEG, PAST>(rows, run, t.dim, l, w[u], sum, scale);
              if (l == 0) t.state[run] = RowState{acc, t.sync_epoch};
            } else if (run < hwm) {  // started in an earlier chunk, ends here
              a_row = run;
              store_vec<SEG>(s_vec + g * dim4, l, active, sum);
            }
          }
        }
      }
      p0 += kBatch;
    }
    if (after == run && run < hwm) {
      b_row = run;
      b_head = head_in;
    }
  }
  if (threadIdx.x == 0) {
    part_row[2 * (uint64_t)at_tile] = kNoRow;
    part_row[2 * (uint64_t)at_tile + 1] = kNoRow;
  }

  // ---- phase 2: join the chunk partials of runs inside this tile -------------------------------
  // A segmented inclusive scan over the chunks: afterwards `sum` of a chunk whose last run continues is that run's sum
  // from its start in the tile on.  The chunks of a wave by shuffles, then the waves through LDS.  (The group with the
  // first piece of a run walked the chunks that follow, one after the other, before: with a hot row in the tile 256 steps
  // for rows of dim 4, 64 for dim 16.  Whole training steps: 58 K IDs of dim 4 99 -> 58 us, 64 K of dim 8 76 -> 56, 264 K
  // of dim 8 103 -> 79, 2 M of dim 4 240 -> 184, 204 K of dim 16 86 -> 77; from dim 36 on the same.)
  if (b_row == kNoRow) sum.zero();
  __shared__ uint32_t s_flags[kReduceWaves];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const bool joins = a_row != kNoRow && g > 0;  // what it joins is asked for beside the scan
  const E* rows = reinterpret_cast<const E*>(t.rows);
  const Vec w = load_row<E, SEG, PAST>(rows, a_row, t.dim, l, joins && active);
  const float acc = joins ? t.state[a_row].acc : 0.f;
  // bit 0: the run comes from the chunk before those summed so far; bit 1: its head is in the tile
  uint32_t flags = (b_row != kNoRow && !b_head && g > 0 ? 1u : 0u) | (b_head ? 2u : 0u);
  if (__ballot(flags & 1u)) {  // wave-uniform
#pragma unroll
    for (uint32_t d = group; d < 64; d <<= 1) {
      const Vec before = sum.from_up(d);
      const uint32_t flags_before = __shfl_up(flags, d);
      if (lane >= d && (flags & 1u)) {
        sum.add(before);
        flags = flags_before;
      }
    }
  }
  if (lane >= 64 - group) store_vec<SEG>(s_carry + wave * dim4, l, active, sum);
  if (lane == 63) s_flags[wave] = flags;
  __syncthreads();
  if (!__ballot(a_row != kNoRow || b_row != kNoRow)) return;  // no run of this wave crosses a border of its chunks
  Vec prev;  // the same sum of the chunk before this one
  prev.zero();
  uint32_t flags_prev = 0;
  for (uint32_t v = wave; v > 0; --v) {  // (wave-uniform)
    prev.add(load_vec<SEG>(s_carry + (v - 1) * dim4, l, active));
    flags_prev = s_flags[v - 1];
    if (!(flags_prev & 1u)) break;
  }
  if (flags & 1u) {
    sum.add(prev);
    flags = flags_prev;
  }
  if (group < 64) {
    const Vec up = sum.from_up(group);
    const uint32_t flags_up = __shfl_up(flags, group);
    if (lane >= group) {
      prev = up;
      flags_prev = flags_up;
    }
  }
  float4* part4 = reinterpret_cast<float4*>(part);
  if (a_row != kNoRow) {
    prev.add(load_vec<SEG>(s_vec + g * dim4, l, active));  // (nothing comes before the first chunk)
    if (g > 0 && (flags_prev & 2u)) {
      adagrad_row<E, SEG, PAST>(t, a_row, w, acc, prev, active, l, group, lr, eps);
    } else {  // it entered the tile from before
      store_vec<SEG>(part4 + (2 * (uint64_t)at_tile) * dim4, l, active, prev);
      if (l == 0) part_row[2 * (uint64_t)at_tile] = a_row;
    }
  }
  if (g == chunks_here - 1 && b_row != kNoRow) {
    store_vec<SEG>(part4 + (2 * (uint64_t)at_tile + 1) * dim4, l, active, sum);
    if (l == 0) part_row[2 * (uint64_t)at_tile + 1] = b_row | (flags & 2u ? kHeadFlag : 0u);
  }
}

// One block per tile; only the block whose tile holds the head of a border-crossing run works.
// The hottest row's chain of pieces bounds it in small batches, the blocks' own latency in large ones.  All rounds of
// pieces are asked for eight at a time, the last one too, and the groups of a wave are summed by shuffles: 6.8 M pairs
// 11.1 -> 7.7 us, 690 K 9.6 -> 7.8.  Rows that take a whole wave have blocks of 512 threads (98 K pairs of dim 512: 18.6
// us with 256, 12.7 with 512, 14.2 with 1024; the update of 98 K to 1 M pairs with hot rows, dims 512 to 1024, 1 to 6 %
// longer with 256, of evenly spread ones and of dims 132 to 256 the same within 2 %); others 256 (6.8 M pairs: 10.2 with
// 512, 18.4 with 1024).
// (A lane group per tile, and a whole block only for runs over more than seven tiles, took 25-43 us there: small
// tiles have many such runs, one after the other in a block.)
constexpr int kCombineWide = 512;
template <typename E, int SEG, int kBlock>
__global__ __launch_bounds__(kBlock) void combine_kernel(TableView t, uint64_t n_tiles, const float* __restrict__ part,
                                                         const uint32_t* __restrict__ part_row, float lr, float eps,
                                                         uint32_t group_log2) {
  extern __shared__ float4 s_mem[];  // [waves of the block][dim / 4]
  using Vec = RowVec<SEG>;
  const uint64_t c = blockIdx.x;
  const uint32_t head = part_row[2 * c + 1];
  if (head == kNoRow || !(head & kHeadFlag)) return;  // block-uniform
  const uint32_t row = head & ~kHeadFlag;
  // number of tiles after c that lie entirely inside the run: nearly always none; where the first 64 all do, 512
  // are looked at together (a row with a tenth of a batch of 26 M spans 2500 of them)
  const auto full_tiles = [&](uint64_t first) {  // leading tiles among the 64 from `first` on (wave-uniform)
    const uint64_t cc = first + (threadIdx.x & 63);
    const uint64_t m = __ballot(cc < n_tiles && part_row[2 * cc + 1] == row);
    return m == ~0ull ? 64u : (uint32_t)(__ffsll((unsigned long long)~m) - 1);
  };
  uint64_t mid = full_tiles(c + 1);
  for (bool more = mid == 64; more;) {
    constexpr int kLook = 8;
    uint32_t full[kLook];
#pragma unroll
    for (int u = 0; u < kLook; ++u) full[u] = full_tiles(c + 1 + mid + (uint64_t)u * 64);
#pragma unroll
    for (int u = 0; u < kLook; ++u) {
      if (more) mid += full[u];
      more = more && full[u] == 64;
    }
  }
  const uint64_t tail = c + 1 + mid;
  const bool has_tail = tail < n_tiles && part_row[2 * tail] == row;
  const uint64_t pieces = 1 + mid + (has_tail ? 1 : 0);
  const uint32_t group = 1u << group_log2, gpb = (uint32_t)kBlock >> group_log2;
  const uint32_t g = threadIdx.x >> group_log2, l = threadIdx.x & (group - 1u);
  const uint32_t dim4 = t.dim >> 2;
  const bool active = l < dim4;
  const float4* part4 = reinterpret_cast<const float4*>(part);
  const Vec w = load_row<E, SEG, false>(reinterpret_cast<const E*>(t.rows), row, t.dim, l, g == 0 && active);
  const float acc = t.state[row].acc;
  Vec sum;
  sum.zero();
  const auto slot_of = [&](uint64_t p) { return p <= mid ? 2 * (c + p) + 1 : 2 * tail; };
  // (a hot row leaves a piece per tile: eight of them in flight)
  constexpr int kPieces = 8 / SEG;
  for (uint64_t p0 = g; p0 < pieces; p0 += (uint64_t)gpb * kPieces) {
    Vec v[kPieces];
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const uint64_t p = p0 + (uint64_t)gpb * u;
      v[u] = load_vec<SEG>(part4 + slot_of(p < pieces ? p : 0) * dim4, l, active && p < pieces);
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u) sum.add(v[u]);
  }
  // the groups of a wave, then the waves
  for (uint32_t d = group; d < 64; d <<= 1) sum.add_xor(d);
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63, groups_per_wave = 64u >> group_log2;
  const uint32_t used = pieces < gpb ? ((uint32_t)pieces + groups_per_wave - 1) / groups_per_wave : kBlock / 64;
  if (wave < used && lane < group) store_vec<SEG>(s_mem + wave * dim4, l, active, sum);
  __syncthreads();
  if (g == 0) {
    Vec total;
    total.zero();
    for (uint32_t q = 0; q < used; ++q) total.add(load_vec<SEG>(s_mem + q * dim4, l, active));
    adagrad_row<E, SEG, false>(t, row, w, acc, total, active, l, group, lr, eps);
  }
}

// The order is worth its launch, 6 to 19 us, where the gradients are more than the caches hold, several occurrences share
// one, and there are a gigabyte or more of them to be read.  Updates without and with it, us: 26 M pairs of 5.2 M bags of dim
// 64 2000 / 1865, 4.2 M of 1 M bags of dim 64 372 / 361 and of dim 128 636 / 596, 1.2 M of 131 K bags of dim 1024 1100 / 1025,
// 25 M of 8.4 M bags of dim 16 965 / 890 (all Zipf 1.1 to 1.2); with half a gigabyte to be read, 0.5 M of 262 K bags of dim
// 256 218 / 228, 2.1 M of 1 M bags of dim 64 241 / 238; where no row is hot 8.4 M of 2.1 M bags of dim 64 925 / 930.
inline bool orders_tiles(uint64_t n, uint64_t n_bags, uint32_t dim) {
  const uint64_t row = dim * sizeof(float);
  return n_bags * row >= kRowsCached && n >= 2 * n_bags && n * row >= 4 * kRowsCached;
}

hipError_t launch_apply_grad_adagrad(const TableView& t, const UpdateWorkspace& ws, const int32_t* d_rows, uint64_t n,
                                     const int64_t* d_offsets, uint64_t n_bags, const float* d_grad, float lr, float eps,
                                     uint32_t hwm_bound, hipStream_t stream, Profiler* prof) {
  if (n == 0 || n_bags == 0) return hipSuccess;
  uint32_t launched = 1, max_bits = 0;
  const hipError_t e =
      sorts_in_one_block(n, n_bags) ? launch_sort_small(t, ws, d_rows, n, d_offsets, n_bags, stream, prof)
      : n <= kSplitMost ? launch_split_pairs(t, ws, d_rows, n, d_offsets, n_bags, stream, prof)
                        : launch_sort_pairs(t, ws, d_rows, n, d_offsets, n_bags, hwm_bound, &launched, &max_bits, stream, prof);
  if (e != hipSuccess) return e;
  uint32_t group_log2 = 0;
  while (group_log2 < 6 && (4u << group_log2) < t.dim) ++group_log2;
  const uint32_t seg = t.dim > 256 ? t.dim / 256 : 1;  // pieces of four elements per lane
  const uint32_t gpb = 256u >> group_log2;
  uint32_t tile = reduce_tile(n, gpb);
  while (tile < kReduceTile && (n + tile - 1) / tile > ws.tiles) tile <<= 1;
  const uint64_t n_tiles = (n + tile - 1) / tile;
  if (n_tiles > ws.tiles) return hipErrorInvalidValue;  // (cannot happen: the workspace is made for this rule)
  const dim3 block(256), grid((unsigned)n_tiles);
  const size_t lds_reduce = (gpb + kReduceWaves) * (t.dim / 4) * sizeof(float4) + tile * sizeof(uint2);
  const size_t lds_combine = kCombineWide / 64 * (t.dim / 4) * sizeof(float4);  // (enough for either block)
  // (see order_tiles_kernel; the sort's counters are free by now, and many more than two words a tile)
  uint32_t* order = nullptr;
  if (orders_tiles(n, n_bags, t.dim)) {
    order = ws.hist + n_tiles;
    MONO_LAUNCH(prof, K_ORDER_TILES, stream, order_tiles_kernel, dim3((unsigned)((n_tiles + kOrderThreads - 1) / kOrderThreads)),
                dim3(kOrderThreads), t.ctl, ws.pair_a, ws.pair_b, (uint32_t)n_tiles, tile, n_bags, launched, max_bits, ws.hist,
                order);
  }
#define MONO_SEG_REDUCE_AS(E, GLOG, SEG, PAST, FEW)                                                                   \
  MONO_LAUNCH_SMEM(prof, K_SEG_REDUCE, stream, (seg_reduce_kernel<E, GLOG, SEG, PAST, FEW>), grid, block, lds_reduce, t, \
                   ws.pair_a, ws.pair_b, n, d_grad, lr, eps, ws.part, ws.part_row, tile, launched, max_bits, order)
#define MONO_SEG_REDUCE(E, GLOG, SEG)                                       \
  if (n * t.dim * sizeof(E) > kRowsCached) {                                \
    MONO_SEG_REDUCE_AS(E, GLOG, SEG, true, false);                          \
  } else if (n_tiles <= kReduceFew) {                                       \
    MONO_SEG_REDUCE_AS(E, GLOG, SEG, false, (SEG == 1 && GLOG >= 3));       \
  } else {                                                                  \
    MONO_SEG_REDUCE_AS(E, GLOG, SEG, false, false);                         \
  }
#define MONO_COMBINE(E, SEG, BLOCK)                                                                                     \
  MONO_LAUNCH_SMEM(prof, K_COMBINE, stream, (combine_kernel<E, SEG, BLOCK>), grid, dim3(BLOCK), lds_combine, t, n_tiles, \
                   ws.part, ws.part_row, lr, eps, group_log2)
#define MONO_SEG_REDUCE_ALL(E)                                          \
  switch (seg) {                                                        \
    case 2: MONO_SEG_REDUCE(E, 6, 2); MONO_COMBINE(E, 2, kCombineWide); break; \
    case 3: MONO_SEG_REDUCE(E, 6, 3); MONO_COMBINE(E, 3, kCombineWide); break; \
    case 4: MONO_SEG_REDUCE(E, 6, 4); MONO_COMBINE(E, 4, kCombineWide); break; \
    default:                                                            \
      switch (group_log2) {                                             \
        case 0: MONO_SEG_REDUCE(E, 0, 1); break;                        \
        case 1: MONO_SEG_REDUCE(E, 1, 1); break;                        \
        case 2: MONO_SEG_REDUCE(E, 2, 1); break;                        \
        case 3: MONO_SEG_REDUCE(E, 3, 1); break;                        \
        case 4: MONO_SEG_REDUCE(E, 4, 1); break;                        \
        case 5: MONO_SEG_REDUCE(E, 5, 1); break;                        \
        default: MONO_SEG_REDUCE(E, 6, 1); break;                       \
      }                                                                 \
      if (group_log2 == 6) {                                            \
        MONO_COMBINE(E, 1, kCombineWide);                               \
      } else {                                                          \
        MONO_COMBINE(E, 1, 256);                                        \
      }                                                                 \
  }
  if (t.bf16) {
    MONO_SEG_REDUCE_ALL(uint16_t)
  } else {
    MONO_SEG_REDUCE_ALL(float)
  }
#undef MONO_COMBINE
#undef MONO_SEG_REDUCE_ALL
#undef MONO_SEG_REDUCE
#undef MONO_SEG_REDUCE_AS
  return hipGetLastError();
}

}  // namespace mono
