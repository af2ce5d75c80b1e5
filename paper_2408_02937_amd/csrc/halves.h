// What host and device agree on about the scan of the halves beside float lists.  Plain C++ but for the three words in front of the
// functions, so that a host compiler can be given this file alone.
#pragma once
#include <cmath>
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

// power of two that brings a query of squared norm qn to a length of 2^13 to 2^14
__host__ __device__ inline float half_piece_scale(float qn) {
  if (!(qn > 0.f) || !(qn < __builtin_inff())) return 1.f;
  const int e = (int)((__builtin_bit_cast(uint32_t, qn) >> 23) & 255u) - 127;  // |q| < 2^((e + 1) / 2)
  int s = 14 - ((e + 2) >> 1);
  s = s > 100 ? 100 : s < -100 ? -100 : s;
  return __builtin_bit_cast(float, (uint32_t)(s + 127) << 23);
}
// ... of a query read by its halves, of squared norm nsq (a short query's squares are not for 32 bits: 1e-23 and shorter is nothing
// there, and what its halves leave out long before)
__host__ __device__ inline float half_query_scale(double nsq) {
  return nsq < 0x1p-60 ? half_piece_scale((float)(nsq * 0x1p100)) * 0x1p50f : half_piece_scale((float)nsq);
}

// ---- scores from the halves beside the lists.  With x' the vector and q' the query as their halves have them (u = 2^-11 the
// unit roundoff of halves, t = 2^-14 sqrt(d) / scale what zeroed subnormals can come to, s = |q - q'| computed),
//   |x - x'| <= u |x| + t.
// Squared distances: | |q - x| - |q' - x'| | <= s + t + u |x|, where |x| is at most |q| plus the distance: whichever of the two
// distances is r, the other one is at most r + 1.001 u (|q| + r) + e with e = s + 1.001 t.  The scan has |q' - x'|^2 in the
// norm form.  Its sum of products is one of at most 64 after the other, each an addition that may be 2^-23 off, and of d / 64 such
// sums; |x'|^2 is of lanes' sums of a quarter of the coordinates: with P >= |q'|, |x'|, all in all it is off by at most
// halves_slack(d) P^2, and the direct form by d + 2 roundings of itself.  (The margin goes with the distance times the norm over
// 2^11, and with the norm squared over 2^15: that of the norm form in one sum of d, which it need not be here, over 2^12 at d 256.)
// Inner products: |<q, x> - <q', x'>| <= |x'| (s + 1.001 u |q|) + 1.001 t |q|, and the roundings of the sum of products and the d
// of the direct one: a |x'| + e.  The scan has |x'| of every vector and keeps the least the inner product's negative can be but
// for e, which is in the bound.
struct HalfQuery {
  float unscale;  // turns a product of halves into a product
  float a;        // squared distances: |q'|^2; inner products: a as above
  float norm;     // |q|, from above
  float e;
  float u;        // 1.001 2^-11, or 0 where the halves of all vectors are their floats
};
// inv: one over the scale of the query's halves, its sign set where nothing is left out of any vector's; qsq: |q'|^2; norm: |q| from above;
// left: s; ixs: one over the scale of the halves beside the lists
__host__ __device__ inline HalfQuery half_query_of(float inv, float qsq, float norm, float left, int d, int metric, float ixs) {
  const bool exact = inv < 0.f;
  const float t = exact ? 0.f : 6.11e-5f * sqrtf((float)d) * ixs;  // (6.11e-5: 1.001 2^-14)
  HalfQuery m{fabsf(inv) * ixs, qsq, norm, left + t, exact ? 0.f : 4.888e-4f};
  if (metric != 0) {
    m.a = 1.002f * (left + norm * (m.u + (float)(d + d / 64 + 140) * 6.0e-8f));
    m.e = 1.002f * t * norm + 1e-30f;
  }
  return m;
}
__host__ __device__ inline float halves_slack(int d) { return (float)(2 * (128 + d / 64 + 1) + 16 * ((d + 31) / 32) + 8) * 6.0e-8f; }
// Squared distances: how far the other one may be where one of the two is v.
__host__ __device__ inline float halves_reach(float v, int d, const HalfQuery &m) {
  const float r0 = sqrtf(fmaxf(v, 0.f)), p = 1.01f * (m.norm + r0) + m.e, fp = halves_slack(d) * p * p;
  float r = sqrtf(r0 * r0 * (1.f + (float)(d + 8) * 6.0e-8f) + fp) * 1.000001f;
  r += m.u * (m.norm + r) + m.e;
  return (r * r + fp) * 1.000001f + 1e-30f;
}
// Negated inner products: what the scan may have kept of a vector whose own is v or better.
__host__ __device__ inline float halves_reach_ip(float v, const HalfQuery &m) { return v + m.e + (fabsf(v) + m.e) * 2.4e-7f; }
// A sample's score v is of the query against what a vector's halves hold.  Squared distances: the vector itself is no further away
// than this; inner products: halves_over times |x'| on top makes it no less than the vector's own, but for e.
__host__ __device__ inline float halves_sampled(float v, int d, const HalfQuery &m) {
  float r = sqrtf(fmaxf(v, 0.f)) * (1.f + (float)(d + 8) * 6.0e-8f);
  r += m.u * (m.norm + r) + m.e;
  return r * r * 1.000001f;
}
__host__ __device__ inline float halves_over(float norm, bool exact, int d) {
  return norm * ((exact ? 0.f : 4.9e-4f) + (float)(2 * d + 8) * 6.0e-8f);
}

}  // namespace rtams
