// Device functions that the sorts of pairs and of exported keys share.
#pragma once

#include "common.h"

namespace mono {

// Lanes of the wave that hold the same digit (below 1 << kBits) as this lane, among the lanes with valid == true.
// Four vector instructions a bit: the bit as a mask, the vote, and both halves of `peers & ~(vote ^ mask)`.  No branch on the
// width in use: the bits above it are zero in all lanes and change nothing.  (Eight instructions a bit, branches between
// them, made up half of the scatter kernel's, and vector units were busy 60 to 87 % of its time.)
template <uint32_t kBits>
__device__ inline uint64_t same_digit_lanes(uint32_t digit, bool valid) {
  constexpr uint32_t kBothOrNeither = 0x90;  // a & ~(b ^ c), bit 4 a + 2 b + c of the table
  const uint64_t all = __ballot(valid);
  uint32_t low = (uint32_t)all, high = (uint32_t)(all >> 32);
#pragma unroll
  for (uint32_t b = 0; b < kBits; ++b) {
    uint32_t mask = (uint32_t)__builtin_amdgcn_sbfe((int)digit, b, 1);
    __asm__("" : "+v"(mask));  // (else the vote takes the bit from the digit again, with a shift of its own)
    const uint64_t vote = __ballot(mask != 0);
    low = __builtin_amdgcn_bitop3_b32(low, (uint32_t)vote, mask, kBothOrNeither);
    high = __builtin_amdgcn_bitop3_b32(high, (uint32_t)(vote >> 32), mask, kBothOrNeither);
  }
  return (uint64_t)high << 32 | low;
}

// How many of these lanes come before this one.
__device__ inline uint32_t lanes_before(uint64_t lanes) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
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
