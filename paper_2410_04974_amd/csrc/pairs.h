// Counting (tile, entry) pairs past 32 bits: a call's total can reach 2^52
// (2^30 entries of up to 2^22 tiles), and one that wrapped would look as if it
// fitted the pair buffers.  Workgroups add saturated sums, the partial sums are
// 64 bits wide, and the total the stage goes by stays at its largest value.
#pragma once

#include <stdint.h>

namespace sixdgs {

constexpr uint32_t kPairsMax = 0xFFFFFFFFu;  // this many pairs or more

__host__ __device__ inline uint32_t add_sat(uint32_t a, uint32_t b) {
  const uint32_t c = a + b;
  return c < a ? kPairsMax : c;
}

__host__ __device__ inline uint32_t pair_total(uint64_t sum) { return sum < kPairsMax ? (uint32_t)sum : kPairsMax; }

// A tile's [first, end) from the pairs before it and its own, inside a buffer
// of cap pairs whatever the counts say; (0, 0) if there are none.
struct PairRange {
  uint32_t first, end;
};
__host__ __device__ inline PairRange pair_range(uint32_t before, uint32_t own, uint32_t cap) {
  const uint32_t first = before < cap ? before : cap;
  const uint32_t end = add_sat(before, own) < cap ? before + own : cap;
  return first < end ? PairRange{first, end} : PairRange{0u, 0u};
}

}  // namespace sixdgs
