// What host and device agree on about the scan of the halves beside float lists.  Plain C++ but for the three words in front of the
// functions, so that a host compiler can be given this file alone.
#pragma once
#include <cstdint>

namespace rtams {

constexpr uint32_t kHalfUnit = 32;  // vectors a wavefront of that scan takes at a time

// Scans of halves: the pairs of an item (32 at most; never 0 where it has any), and behind six bits the units its segment has
// by the length the plan saw.  A scan goes no further, whatever an insertion has published since: the block table past that
// length may lie in this kernel's caches as it was before its entries were made.  (A segment of 2^17 units is the
// longest the plan makes.)
__host__ __device__ inline uint32_t half_item_word(uint32_t pairs, uint32_t len, uint32_t segment, uint32_t seg_groups) {
  const uint32_t per = seg_groups * (64 / kHalfUnit), units = len / kHalfUnit + (len % kHalfUnit ? 1u : 0u), first = segment * per;
  const uint32_t mine = units > first ? units - first : 0u;
  return pairs | (mine < per ? mine : per) << 6;
}
__host__ __device__ inline uint32_t half_item_pairs(uint32_t word) { return word & 63u; }
__host__ __device__ inline uint32_t half_item_units(uint32_t word) { return word >> 6; }

}  // namespace rtams
