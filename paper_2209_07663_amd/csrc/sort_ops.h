// Device functions that the kernels of the pair sort share.
#pragma once

#include "common.h"

namespace mono {

// Lanes of the wave that hold the same digit (of `bits` <= kBits bits) as this lane, among the lanes with valid == true.
template <uint32_t kBits>
__device__ inline uint64_t same_digit_lanes(uint32_t digit, uint32_t bits, bool valid) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (uint32_t b = 0; b < kBits; ++b) {
    if (b < bits) {  // wave-uniform
      const bool bit = (digit >> b) & 1u;
      const uint64_t vote = __ballot(bit);
      peers &= bit ? vote : ~vote;
    }
  }
  return peers;
}

// key of occurrence i in pass 0: its row, or hwm if the occurrence was dropped
__device__ inline uint32_t first_key(const int32_t* rows, uint64_t i, uint32_t hwm) {
  const uint32_t r = (uint32_t)rows[i];
  return r < hwm ? r : hwm;
}

// An offset of the caller's, bounded to the n occurrences of the batch.
__device__ inline uint64_t bounded_offset(const int64_t* offsets, uint64_t b, uint64_t n) {
  const int64_t o = offsets[b];
  return o < 0 ? 0ull : ((uint64_t)o > n ? n : (uint64_t)o);
}

}  // namespace mono
