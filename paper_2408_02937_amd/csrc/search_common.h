// What the kernels of the search path share: monotone key maps, where a query's survivor records
// lie, workgroup-wide selection and sorting in LDS, the fp32 score of a vector against a query,
// and the launch shape of the list scan (the planning kernel needs it as well).
#pragma once
#include <type_traits>
#include "halves.h"
#include "rtams_launch.h"

namespace rtams {

// ------------------------------------------------------------------ key maps
// Monotone maps from scores to unsigned keys: a smaller key is a better score.
__device__ inline uint64_t key_of_double(double x) {
  uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ inline uint32_t key_of_float(float x) {
  uint32_t b = __float_as_uint(x);
  return (b >> 31) ? ~b : (b | 0x80000000u);
}

// ------------------------------------------------------- survivor records
// How many a query has.  Every wavefront of the scan reserves places from these counters, and reservations on one
// cache line are served one after the other, whichever queries they are for: each counter has a line to itself.
// (They lie in the room of the exact coarse scores, which nobody reads any more once the probes are chosen.)
__device__ inline uint32_t *rec_count(const SearchScratch &S, uint32_t q) { return S.rec_cnt + ((size_t)q << S.rec_shift); }
// Where a query's records lie: in its request's slice or, flagged, in the reserve all resources share.
__device__ inline uint32_t *rec_keys_of(const SearchScratch &S, unsigned long long qbase) {
  return (qbase & kInOverflow) ? S.ovf_key + (qbase & ~kInOverflow) : S.rec_key + qbase;
}
__device__ inline uint32_t *rec_poss_of(const SearchScratch &S, unsigned long long qbase) {
  return (qbase & kInOverflow) ? S.ovf_pos + (qbase & ~kInOverflow) : S.rec_pos + qbase;
}
// Room for `want` entries in the request's chunk of the shared reserve (called by one thread per
// query): the start, flagged, or ~0.  The first query of a request that needs it leases a free chunk
// and installs it for the request; one that loses that race to a sibling hands its chunk straight
// back and shares the sibling's.  Nobody waits for anybody beyond a few bounded second looks.
__device__ inline unsigned long long overflow_take(const SearchScratch &S, unsigned long long want) {
  if (S.ovf_chunks == 0 || want > S.ovf_chunk_cap) return ~0ull;
  // Siblings that race for the request's chunk may hold several free chunks between them for a moment
  // (all but one are handed back at once), and a query of ANOTHER request that looks just then finds
  // every chunk out although one is about to come back: it looks again a bounded number of times
  // before it gives up (a chunk that stays out is held by a request for as long as that request runs).
  uint32_t c = __hip_atomic_load(S.req_chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int round = 0; round < 32 && c == 0; ++round) {
    for (uint32_t e = 0; e < S.ovf_chunks && c == 0; ++e)
      if (atomicCAS(&S.ovf_leased[e], 0u, 1u) == 0u) {
        const uint32_t seen = atomicCAS(S.req_chunk, 0u, e + 1u);
        if (seen == 0u) c = e + 1u;
        else { atomicExch(&S.ovf_leased[e], 0u); c = seen; }
      }
    if (c == 0) c = __hip_atomic_load(S.req_chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // a sibling may have got the last one
    if (c == 0) __builtin_amdgcn_s_sleep(32);
  }
  if (c == 0) return ~0ull;  // every chunk is out
  const unsigned long long off = atomicAdd(S.req_cursor, want);
  if (off + want > S.ovf_chunk_cap) return ~0ull;
  return kInOverflow | ((unsigned long long)(c - 1u) * S.ovf_chunk_cap + off);
}
// Every selection workgroup of a request reports here when it has read its last record; the last
// one returns the request's chunk, if it holds one, and resets the request's words.
__device__ inline void overflow_request_done(const SearchScratch &S, uint32_t workgroups) {
  if (S.ovf_chunks == 0) return;
  __threadfence();
  if (atomicAdd(S.req_done, 1u) + 1u != workgroups) return;
  const uint32_t c = __hip_atomic_load(S.req_chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(S.req_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(S.req_cursor, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (c) {
    __hip_atomic_store(S.req_chunk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();
    atomicExch(&S.ovf_leased[c - 1u], 0u);
  }
}

// ------------------------------------------------- workgroup radix selection
// Finds the threshold of the k smallest keys among the valid items 0..n-1.
// fn(i, key) returns false for items that do not take part.  On return T is
// a threshold such that every key < T belongs to the k smallest and, of the
// c_eq keys not yet told apart from T, `need` belong to them (when c_eq == need
// the selection stops early and T is the largest key that group can hold; else
// T is the k-th smallest key itself and the c_eq keys equal it).  Callers take
// key < T, and key == T under the tie rule.  Requires 1 <= k <= #valid.
// `stop`: the caller is content with a threshold that admits at most so many keys (k - need + c_eq of them, all
// <= T): it sorts what it takes anyway, and the passes that would tell the last bin's few keys apart, each with two
// barriers and a microsecond of its own, are left out.
struct SelectResult {
  uint64_t T;
  uint32_t need, c_eq;
};

// After a histogram pass: the first wavefront finds the bin that holds the
// need-th smallest item; bc = {bin, items in lower bins, items in the bin}.
__device__ inline void wg_pick_bin(const uint32_t *hist, uint32_t need, uint32_t *bc) {
  if (threadIdx.x < kWave) {  // first wavefront: which bin holds the need-th item
      int l = threadIdx.x;
      uint32_t h0 = hist[4 * l], h1 = hist[4 * l + 1], h2 = hist[4 * l + 2], h3 = hist[4 * l + 3];
      uint32_t sum = h0 + h1 + h2 + h3, incl = wave_running_sum(sum);
      uint32_t excl = incl - sum;
      if (excl < need && need <= incl) {  // exactly one lane
        uint32_t cum = excl;
        int dg;
        uint32_t hh;
        if (cum + h0 >= need) { dg = 0; hh = h0; }
        else { cum += h0;
          if (cum + h1 >= need) { dg = 1; hh = h1; }
          else { cum += h1;
            if (cum + h2 >= need) { dg = 2; hh = h2; }
            else { cum += h2; dg = 3; hh = h3; } } }
        bc[0] = (uint32_t)(4 * l + dg);
        bc[1] = cum;
        bc[2] = hh;
      }
    }
    __syncthreads();
}

// LDS of a selection: two histograms of 256 bins (while one is filled the other is cleared for the
// next pass) and a slot of two 64-bit words per wavefront for the range of the keys.
constexpr int kSelectLdsWords = 2 * 256 + 4 * 16;

// `each(body)` calls body(key) for every key of the calling thread that takes part.  `hist` holds
// kSelectLdsWords words, 8-byte aligned; the workgroup has at most 16 wavefronts.
template <int BITS, typename Each>
__device__ __forceinline__ SelectResult wg_radix_select_each(uint32_t k, Each each, uint32_t *hist, uint32_t *bc, uint32_t stop = 0) {
  typedef typename std::conditional<BITS == 32, unsigned int, unsigned long long>::type Key;  // what the range is reduced in
  // The first digit is the 8 bits that end at the highest bit in which any two keys differ: scores
  // of one query's candidates share sign, exponent and often the first mantissa bits; digits on
  // which every key agrees would make all lanes hit one LDS word (which serialises completely) and
  // decide nothing, and a first digit cut out at a byte boundary often tells only a handful of
  // bins apart.  This way the first pass uses all 256 bins, and a few hundred keys are usually
  // done after one or two.
  uint64_t *range = reinterpret_cast<uint64_t *>(hist + 512);  // per wavefront: {min, max}
  const int lane = (int)(threadIdx.x & (kWave - 1)), wave = (int)(threadIdx.x / kWave);
  __syncthreads();  // whatever used this LDS before is done
  for (int b = threadIdx.x; b < 256; b += blockDim.x) hist[b] = 0;
  {
    Key lo = ~(Key)0, hi = 0;
    each([&](uint64_t key) { lo = (Key)key < lo ? (Key)key : lo; hi = (Key)key > hi ? (Key)key : hi; });
    lo = wave_reduce_last(lo, [](Key a, Key b) { return b < a ? b : a; });
    hi = wave_reduce_last(hi, [](Key a, Key b) { return b > a ? b : a; });
    int at = lane;
    asm volatile("" : "+v"(at));  // (no mask of these lanes is kept in scalar registers, which the callers have none to spare of)
    if (at == kWave - 1) { range[2 * wave] = (uint64_t)lo; range[2 * wave + 1] = (uint64_t)hi; }
  }
  __syncthreads();
  uint64_t kmin = ~0ull, kmax = 0ull;
  for (int w0 = 0; w0 < (int)(blockDim.x / kWave); w0 += 4) {  // (workgroups of this library have whole fours of wavefronts)
#pragma unroll
    for (int w = w0; w < w0 + 4; ++w) {
      const uint64_t a = range[2 * w], b = range[2 * w + 1];
      kmin = a < kmin ? a : kmin;
      kmax = b > kmax ? b : kmax;
    }
  }
  int shift = 0;
  uint64_t prefix = 0, mask = 0;
  {
    const uint64_t diff = kmin ^ kmax;
    const int top = diff ? 63 - __clzll((long long)diff) : -1;  // highest bit in which keys differ
    shift = top < 7 ? 0 : top - 7;
    if (shift > BITS - 8) shift = BITS - 8;
    if (shift + 8 < 64) {
      mask = ~0ull << (shift + 8);
      if (BITS < 64) mask &= (1ull << BITS) - 1ull;
    }
    prefix = kmax & mask;
  }
  uint32_t need = k, c_eq = 0;
  uint32_t *cur = hist, *other = hist + 256;
  for (;;) {
    each([&](uint64_t key) {
      if ((key & mask) == prefix) atomicAdd(&cur[(uint32_t)(key >> shift) & 255u], 1u);
    });
    for (int b = threadIdx.x; b < 256; b += blockDim.x) other[b] = 0;  // for the next pass; last read before the previous barrier
    __syncthreads();
    wg_pick_bin(cur, need, bc);  // ends with a barrier
    const uint32_t dg = bc[0];  // (bc is written again only behind the next barrier)
    need -= bc[1];
    c_eq = bc[2];
    // A digit that overlaps the one before it (the last one, when fewer than 8 bits were left) repeats
    // bits the prefix already holds: only keys that match the prefix were counted, so they agree.
    prefix |= (uint64_t)dg << shift;
    mask |= (uint64_t)255u << shift;
    if (c_eq == need || k - need + c_eq <= stop) {  // the whole bin is taken: the lower digits cannot matter
      if (shift > 0) prefix |= (1ull << shift) - 1ull;  // threshold = largest key of the bin
      break;
    }
    if (shift == 0) break;
    shift = shift >= 8 ? shift - 8 : 0;
    uint32_t *t = cur; cur = other; other = t;
  }
  return {prefix, need, c_eq};
}

// Items 0..n-1 given by fn(i, key) (false: the item does not take part); keys are
// read from memory, four independent loads in flight per thread.
template <int BITS, typename Fn>
__device__ __forceinline__ SelectResult wg_radix_select(int n, uint32_t k, Fn fn, uint32_t *hist, uint32_t *bc, uint32_t stop = 0) {
  auto each = [&](auto body) {
    for (int i0 = threadIdx.x; i0 < n; i0 += 4 * blockDim.x) {
      uint64_t key[4];
      bool ok[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // clamped index: the loads are unconditional and issue back to back
        const int i = i0 + u * (int)blockDim.x;
        ok[u] = fn(i < n ? i : n - 1, key[u]) && i < n;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (ok[u]) body(key[u]);
    }
  };
  return wg_radix_select_each<BITS>(k, each, hist, bc, stop);
}

// Bitonic sort of m (power of two) entries in LDS by (k1, k2) ascending; pay is carried along.  A wavefront takes 64
// neighbouring pairs: with strides up to 64 they lie in 128 entries that are its own, and as LDS operations of one
// wavefront execute in order those steps need no barrier; only the longer strides have one in front and one behind.
// (One wavefront for all of it took 35 us for the 293 finalists of a hot list's query; this takes 5.)
__device__ inline void wg_bitonic_sort(int m, uint64_t *k1, uint64_t *k2, uint32_t *pay) {
  __syncthreads();
  for (int size = 2; size <= m; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride > kWave) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      for (int t = threadIdx.x; t < m / 2; t += (int)blockDim.x) {
        const int i = 2 * t - (t & (stride - 1)), j = i + stride;
        const bool up = (i & size) == 0;
        const uint64_t a1 = k1[i], a2 = k2[i], b1 = k1[j], b2 = k2[j];
        const bool a_gt_b = a1 != b1 ? a1 > b1 : a2 > b2;
        if (a_gt_b == up) {
          k1[i] = b1; k2[i] = b2; k1[j] = a1; k2[j] = a2;
          const uint32_t p = pay[i]; pay[i] = pay[j]; pay[j] = p;
        }
      }
      if (stride > kWave) __syncthreads();
    }
  }
  __syncthreads();
}

__device__ inline int next_pow2(int v) {
  int m = 1;
  while (m < v) m <<= 1;
  return m;
}

// Sort of the first n entries in LDS by (k1, k2) ascending, pay carried along; entries from n up to
// the next power of two may be overwritten.  A few hundred entries at most are ranked: a group
// of S neighbouring lanes counts, each over its share of the entries, how many come before entry
// e (equal pairs in the order they stand in), and the entry is written to that place — two
// barriers instead of the dozens of dependent LDS round trips of a sorting network, which costs a
// single wavefront 5 to 7 us for 32 to 128 entries.  More entries go through the network.
// BITS: what the first key has, 32 or 64.
constexpr int kRankSortMax = 256;
template <int BITS>
__device__ inline void wg_sort(int n, uint64_t *k1, uint64_t *k2, uint32_t *pay) {
  const int T = (int)blockDim.x;
  if (n > kRankSortMax || n > T) {  // uniform over the workgroup
    const int m = next_pow2(n > 0 ? n : 1);
    __syncthreads();
    for (int p = n + (int)threadIdx.x; p < m; p += T) { k1[p] = ~0ull; k2[p] = ~0ull; pay[p] = 0; }
    wg_bitonic_sort(m, k1, k2, pay);
    return;
  }
  __syncthreads();
  int S = 1;  // lanes per entry: a power of two, at most a wavefront, S * n <= T
  while (S < kWave && 2 * S * n <= T) S *= 2;
  const int e = (int)threadIdx.x / S, s = (int)threadIdx.x % S;
  const bool on = e < n;
  uint64_t a1 = 0, a2 = 0;
  uint32_t ap = 0, before = 0;
  if (on) {
    a1 = k1[e]; a2 = k2[e]; ap = pay[e];
    const int per = (n + S - 1) / S;
    const int lo = s * per, hi = lo + per < n ? lo + per : n;
    // 32 bits decide nearly always (64-bit comparisons take four times as long): the whole key, or the upper half of
    // it.  Everything else is looked at only where those are equal, other than for the entry itself, which every entry
    // meets (it made nearly every turn of some lane a trip to LDS for the second key: 100 entries took 2.9 us).
    const uint32_t *w = reinterpret_cast<const uint32_t *>(k1) + (BITS == 64 ? 1 : 0);
    const uint32_t aw = w[2 * e];
    auto count = [&](int j, uint32_t bw) {
      before += bw < aw ? 1u : 0u;
      if (bw == aw && j != e) {
        const uint64_t b1 = k1[j], b2 = k2[j];
        before += (b1 < a1 || (b1 == a1 && (b2 < a2 || (b2 == a2 && j < e)))) ? 1u : 0u;
      }
    };
    int j = lo;
    for (; j + 4 <= hi; j += 4) {
      const uint32_t b0 = w[2 * j], b1 = w[2 * j + 2], b2 = w[2 * j + 4], b3 = w[2 * j + 6];
      count(j, b0); count(j + 1, b1); count(j + 2, b2); count(j + 3, b3);
    }
    for (; j < hi; ++j) count(j, w[2 * j]);
  }
  before = group_sum(before, S);  // the S lanes of an entry are neighbours in one wavefront
  __syncthreads();  // everybody has read
  if (on && s == 0) { k1[before] = a1; k2[before] = a2; pay[before] = ap; }
  __syncthreads();
}


// ------------------------------------------------------------------ fp32 score
// Score of one vector against one query, 4 dimensions at a time, one FMA chain
// in the order of the dimensions.
typedef __attribute__((address_space(1))) float GlobalFloat;
typedef __attribute__((address_space(1))) uint32_t GlobalU32;

template <int METRIC>
__device__ __forceinline__ void accumulate(float &acc, const float4 &x, const float4 &y) {
  if (METRIC == 0) {
    const float t0 = x.x - y.x, t1 = x.y - y.y, t2 = x.z - y.z, t3 = x.w - y.w;
    acc = fmaf(t0, t0, acc); acc = fmaf(t1, t1, acc); acc = fmaf(t2, t2, acc); acc = fmaf(t3, t3, acc);
  } else {
    acc = fmaf(x.x, y.x, acc); acc = fmaf(x.y, y.y, acc); acc = fmaf(x.z, y.z, acc); acc = fmaf(x.w, y.w, acc);
  }
}

// ------------------------------------------- dot products on the matrix cores
// v_mfma_f32_4x4x1 (16 blocks): a wavefront multiplies, block by block, a column of 4 values of A by a
// row of 4 values of B.  Lane l supplies one value of each; component r of the result in lane l is
//   a[lane 4 (l / 4) + r] * b[lane l]
// added to what the component held.  With a = one coordinate of the 64 vectors of a group (lane =
// vector, exactly what the interleaved layout hands to a wavefront) and b = the same coordinate of
// query l % 4, d such instructions leave, in lane l, the inner products of vectors 4 (l / 4) .. + 3 with
// query l % 4: 64 vectors x 4 queries per instruction and coordinate, no data movement in between.
typedef float MfmaAcc __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void mfma_step(MfmaAcc &acc, float x, float y) {
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, y, acc, 0, 0, 0);
}
// a chunk of 4 coordinates into one accumulator, in the order of the coordinates
__device__ __forceinline__ void mfma_chunk(MfmaAcc &acc, const float4 &x, const float4 &y) {
  mfma_step(acc, x.x, y.x);
  mfma_step(acc, x.y, y.y);
  mfma_step(acc, x.z, y.z);
  mfma_step(acc, x.w, y.w);
}
// value of lane 4 (l / 4) + r for every lane l (a move inside each group of four lanes)
template <int R>
__device__ __forceinline__ float quad_broadcast(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), R * 0x55, 0xf, 0xf, true));
}

// value of lane 16 (l / 16) + r for every lane l (a move inside each row of sixteen lanes)
template <int R>
__device__ __forceinline__ float row_broadcast(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x150 + R, 0xf, 0xf, true));
}

// ---- norm form of the squared distance.  On the matrix cores a squared distance is scored as
// |x|^2 + |q|^2 - 2 <x, q> (the inner products are the contraction; |x|^2 is accumulated once per
// vector beside it).  That value differs from the direct form sum (x - q)^2 (which is what the bound's
// sample computes and what is returned) by rounding errors that grow with the norms, not with the
// distance:
//   |norm form - direct form| <= slack * (2 v + 3 |q|^2),  slack = 1.01 (4 d + 8) 2^-24,
// for v either of the two values (d roundings for |x|^2, up to 2 d for <x, q> whatever the order of
// its terms, three more for the combination, d + 2 roundings of the direct form; |x|^2 + |q|^2 <=
// 2 |x - q|^2 + 3 |q|^2).  So whoever compares a norm-form score with a limit taken from direct-form
// scores, or the other way round, first raises the limit by that much ("loosened"), and the selection
// scores its finalists again in the direct form: the result is the one the direct form gives.
// Lists of halves and bytes may go through 16-bit matrix instructions with the query in three pieces (scan_mm.hip), which
// may add with roundings either way, 2^-23 each: d of them on the products of the first piece, 2 d on those of the others,
// which are 2^-7 of them at most and are summed for themselves, and d on |x|^2 for halves (none for bytes); with
// |x| |q| <= 1.5 |q|^2 + v / 2 and |x|^2 <= 2 |q|^2 + 2 v that is (10.2 |q|^2 + 7.1 v) d 2^-24 with the direct form's own
// d + 2 roundings: the same margin holds both.
__host__ __device__ inline uint32_t narrow_row_bytes(const Dev &D) {  // of a query's piece in LDS
  return (uint32_t)((D.vchunks + 3) / 4 * 4) * (D.storage == 1 ? 16u : 32u) + 16u;
}
__host__ __device__ inline bool scans_narrow(const Dev &D) { return D.scan_mfma == 2; }
__device__ inline float norm_form_slack(int d) { return 1.01f * (float)(4 * d + 8) * 5.9604645e-8f; }
__device__ inline float loosened(float v, float slack, float qn) {
  const float r = v + slack * (2.f * fmaxf(v, 0.f) + 3.f * qn) + 1e-30f;
  return r + fabsf(r) * 2.4e-7f;  // the rounding of this very computation
}
__device__ inline float l2_score_of_key(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}
__device__ inline uint32_t loosened_key(uint32_t key, float slack, float qn) {
  if (key == 0xFFFFFFFFu) return key;  // "keep everything"
  return key_of_float(loosened(l2_score_of_key(key), slack, qn) + 0.0f);
}
// which lists a request scores through the norm form: flat lists under the L2 metric
__device__ __host__ inline bool uses_norm_form(const Dev &D) {
  return D.scan_mfma != 0 && D.metric == 0 && D.pq_m == 0;
}

// Whether the halves of every vector inserted so far are its floats (then nothing is left out: u and t are zero).  Insertions
// write the word while searches run, so a request asks once, for each query where its bound is set, behind the lengths of its
// lists (an insertion writes the word before it publishes: "yes" holds for all that the request may see), and goes by what it wrote
// down then (halves_exact_for): workgroups that share a query, and the threads of one, have to agree.
__device__ inline bool halves_are_floats(const Dev &D) {
  return __hip_atomic_load(&D.ctrl->half_inexact, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
}
__host__ __device__ inline uint32_t half_row_units(const Dev &D) { return (uint32_t)(D.hchunks + 3) / 4u * 4u; }
// of query q: its halves, zeros up to whole steps of 32 coordinates, then what half_query() makes its HalfQuery of: one over its
// scale (with the sign set where halves_are_floats), |q'|^2, |q| from above, and s (in the room the coarse filter has for
// halves of the queries, twice what they take; nobody needs those once the probes are chosen)
__device__ inline u32x4 *half_query_row(const Dev &D, const SearchScratch &S, uint32_t q) {
  return S.qhalf + (size_t)q * (half_row_units(D) + 1u);
}
__device__ inline bool halves_exact_for(const Dev &D, const SearchScratch &S, uint32_t q) {
  return *reinterpret_cast<const float *>(half_query_row(D, S, q) + half_row_units(D)) < 0.f;
}
__device__ inline HalfQuery half_query(const Dev &D, const SearchScratch &S, uint32_t q) {
  const float4 w = *reinterpret_cast<const float4 *>(half_query_row(D, S, q) + half_row_units(D));
  return half_query_of(w.x, w.y, w.z, w.w, D.d, D.metric, 1.f / halves_scale(D));
}
__device__ inline uint32_t halves_reach_key(const Dev &D, uint32_t key, const HalfQuery &m) {
  const float v = l2_score_of_key(key);
  if (!(v < __builtin_inff())) return 0xFFFFFFFFu;  // "keep everything", as behind a NaN
  const float w = halves_reach(v, D.d, m);
  return w < __builtin_inff() ? key_of_float(w) : 0xFFFFFFFFu;
}
__device__ inline uint32_t halves_reach_ip_key(uint32_t key, const HalfQuery &m) {
  const float w = halves_reach_ip(l2_score_of_key(key), m);
  return fabsf(w) < __builtin_inff() ? key_of_float(w + 0.0f) : 0xFFFFFFFFu;
}
// The query's bound, the k-th best score of a sample of its candidates from their halves, as one of what the scan of halves has.
__device__ inline uint32_t halves_bound_key(const Dev &D, uint32_t key, const HalfQuery &m) {
  if (key == 0xFFFFFFFFu) return key;
  if (D.metric != 0) return halves_reach_ip_key(halves_reach_ip_key(key, m), m);
  const float v = l2_score_of_key(key);
  if (!(v < __builtin_inff())) return 0xFFFFFFFFu;
  return halves_reach_key(D, key_of_float(halves_sampled(v, D.d, m)), m);
}
// A vector or query whose halves are not finite says nothing: it is kept, and its query's flag, behind its counter of records, has
// the selection score all of the records again.
__device__ inline uint32_t *rec_flag(const SearchScratch &S, uint32_t q) { return rec_count(S, q) + 1; }
// ... and behind that what the workgroups that share a query's selection count: those that are done, finalists scored, and whether one of
// them found that it cannot be shared (select.hip)
__device__ inline uint32_t *rec_done(const SearchScratch &S, uint32_t q) { return rec_count(S, q) + 2; }
__device__ inline uint32_t *rec_scored(const SearchScratch &S, uint32_t q) { return rec_count(S, q) + 3; }
__device__ inline uint32_t *rec_alone(const SearchScratch &S, uint32_t q) { return rec_count(S, q) + 4; }
__device__ inline void rec_words_clear(const SearchScratch &S, uint32_t q) {
  uint32_t *w = rec_count(S, q);
#pragma unroll
  for (int i = 0; i < 5; ++i) w[i] = 0u;
}


// ---------------------------------------------------- launch shape of the scan
// Hardware hands consecutive workgroup ids to the 8 XCDs in turn; a workgroup of the scan is up to
// four wavefronts, one work item each.
constexpr uint32_t kXcds = 8;
constexpr int kComputeUnits = 256;
constexpr int kScanWaves = 4;

// Launch shape of a list scan.  Two kernels share the plan of work items (list, segment, tile of the
// queries probing the list):
//  - vector unit: a workgroup is up to four wavefronts that take four consecutive items, one each, every one with its
//    own tile of up to 8 queries in LDS;
//  - matrix cores: a workgroup takes ONE item, its tile of up to 32 queries sits in LDS once, and its four wavefronts
//    share out the item's groups of vectors.  Large tiles are what keeps a hot list from being read once per 8 of the
//    dozens of queries that probe it; the price is registers (3 wavefronts per SIMD in long scans) and a tile to
//    set up per item, which small requests, whose tiles hold a query or two, do not get back
//    (measured at 1 and 32 queries: 15 to 20 % slower than the vector unit with its partial-distance
//    pruning; mm_scan_pays() has the larger ones).
struct ScanShape {
  bool mm;           // a matrix-core kernel
  int tile_q;        // queries of a tile at most
  int seg_base;      // segments are seg_base << choice groups of 64 vectors: 2, or 1 for small requests over short lists
  int min_choice;    // the shortest the plan may choose
  int items_per_wg;  // items a workgroup takes
  int threads;       // of a workgroup
  int grid;          // workgroups
  size_t lds;        // dynamic LDS bytes of a workgroup
};
constexpr int kMmWaves = 4;            // wavefronts of a workgroup of the matrix-core scan
constexpr int kMmTileMax = 32;         // queries of its tile at most
constexpr int kMmQueryWords = 12;      // 32-bit words of LDS per query of a tile beside its coordinates
constexpr int kMmStageCap = 256;       // survivors a wavefront stages in LDS before it reserves their places
constexpr size_t kMmStageBytes = (size_t)kMmStageCap * 9 + 8 * kMmTileMax;  // keys, positions, rows, and two words per query of the tile
constexpr uint32_t kHalfStep = 2048;   // the scan of halves: bytes of a step, and steps a wavefront has in LDS
constexpr uint32_t kHalfRing = 2;
constexpr int kHalfQueryWords = 6;
constexpr int kHalfStageCap = 128;
constexpr size_t kHalfStageBytes = (size_t)kHalfStageCap * 9 + 8 * kMmTileMax;
constexpr int kHalfConsts = 4;         // the scan of halves: 32-bit words per query of a tile that go into its scores
constexpr uint32_t kHalfPlaces = 8;    // ... and the places of a wavefront's groups it keeps (copies are at most four groups ahead)
constexpr size_t kMmLdsMax = 160 * 1024 - 1024;  // what a workgroup may take of the CU's 160 KiB
// The vector unit's scan walks groups singly where lists have so few that pairs leave much of the last one empty, and the
// request has fewer than two groups for every SIMD.  Pairs / one at a time, us a request: 10 k x 32 in lists of 3 groups,
// 10 and 64 queries x 8 probes, 47.2 / 45.6 and 49.5 / 47.0; 0.5 M x 768 in lists of 1, 1 and 8 queries x 32 probes,
// 75.3 / 64.1 and 102.6 / 92.4; but 1 M x 128 in lists of 16, 1 and 2 queries, 60.2 / 61.0 and 63.2 / 64.5, and 12 queries
// (6,100 groups) 80.9 / 86.7.
constexpr int64_t kSingleList = 4;
constexpr int64_t kSingleGroups = 2048;
constexpr int kMmMinBatch = 64;        // queries of a request from which the matrix-core scan pays

// Whether a request of 64 queries or more scans on the matrix cores.  A tile is the queries of the request that probe one
// list, and what speaks for the matrix cores is arithmetic: many queries to a list, or (inner products) so wide vectors
// that the vector unit's tiles of queries in LDS leave a compute unit few wavefronts (from d 512).  What speaks against
// them is the set-up of a workgroup per item, which short lists do not repay.  Requests of 64 to 256 queries were measured
// on both over d 32 to 1536, 64 to 16,384 lists of 100 to 10,000 vectors and a quarter of a pair to 256 pairs to a list,
// even lists and hot ones (16 times the average and more; a good share of any batch probes them).  Vector unit / matrix
// cores, us a request, the products of the request in brackets:
//  inner products, floats, even lists.  d 96, 1,024 lists of 1,000: 142 / 141 (0.8 G), 179 / 149 (1.6 G); of 300: 92 / 112
//    (0.5 G).  d 256, 64 lists of 10,000: 192 / 211 (0.7 G), 272 / 259 (5 G), 1,384 / 1,003 (42 G); 1,024 of 300: 159 / 204
//    (1.3 G).  From d 512 by pairs: d 512, 64 lists of 1,000: 71 / 65 at 1 pair, 433 / 338 at 256; d 768, 8,192 lists of 400:
//    551 / 551 at 1/4 pair, 880 / 1,060 at 1/2, 64 lists of 10,000: 295 / 295 at 1, 5,956 / 3,086 at 256; d 1536: 504 / 494,
//    22,353 / 7,037.  Over all 863 the rule is 1.2 % from the better of the two on average, 1.46 times at worst (d 512,
//    1,024 lists of 300, 16 pairs: 294 / 430)
//  the same, hot lists.  d 256, 16,384 lists of 400: 775 / 852 (3.6 G with the hot one), 1,006 / 940 (8 G); 1,024 of 300:
//    198 / 279 (1.6 G); of 4,000: 1,365 / 1,004 (22 G).  d 768, 4,096 lists of 100: 591 / 768 (1.6 G); of 500: 1,900 / 1,267
//  inner products, halves and bytes.  d 128, 1,024 lists of 300: 98 / 103 (0.6 G), 4,096 of 500 with a hot one 154 / 142
//    (0.3 G); halves, d 384, 64 of 10,000: 130 / 109 (0.3 G), 2,159 / 1,355 (63 G); from d 512 always: halves, d 768, 64
//    lists of 300: 82 / 86, 355 / 231; bytes 96 / 109, 302 / 261
//  squared distances, floats: by their pairs and the hot list alone, also where that costs a tenth: behind the matrix cores
//    the selection scores its finalists again in four short sums, which come out closer to 64 bits (2 to 3 times, at d 256)
//    than the one long sum of the vector unit's scan.  1,024 lists of 977 x 128: 4 pairs to a list 158 / 171, 8 205 / 195,
//    16 281 / 215; lists of 390 x 200: 16 pairs 127 / 134; hot lists, 16,384 of 1,220 x 256: 64 queries 2,000 / 2,190, 128
//    2,620 / 2,510, 256 3,490 / 2,900
//  squared distances, halves and bytes.  1,024 lists of 1,000 x 128, halves: 2 pairs 110 / 110, 4 133 / 126; bytes: 1 pair
//    89 / 92, 2 110 / 103; halves from d 512, where the margin of the norm form admits more finalists: d 768, 4 pairs
//    535 / 626, 8 825 / 802.  Hot lists, halves, 1,024 of 1,000 x 128: 64 queries x 16 probes 124 / 120, 256 x 64 340 / 229;
//    x 768: 550 / 691, 933 / 914 at 128 x 32, 1,933 / 1,298 at 256 x 64; 4,096 of 100 x 64: 88 / 99
inline bool mm_scan_pays(const Dev &D, int64_t nq, int64_t nprobe, int64_t avg_len, int64_t max_len) {
  const int64_t pairs = nq * nprobe, nlist = D.nlist, d = D.d;
  const bool hot = max_len >= 16 * avg_len;
  if (D.metric == 0) {
    if (D.storage == 0) return pairs >= nlist || hot;
    if (hot && avg_len >= 448 && (nq >= 128 || pairs >= nlist)) return true;
    return avg_len >= 512 && pairs >= (D.storage == 2 ? 2 : d >= 512 ? 8 : 4) * nlist;
  }
  // multiply-adds the request can expect, a tenth of its queries meeting the longest list
  const double products = (double)(nq * d) * (double)(nprobe * avg_len + max_len / 10);
  if (D.storage != 0) return d >= 512 || ((avg_len >= 512 || (hot && max_len >= 16384)) && products >= 0.3e9);
  if (hot) return products >= (d >= 512 ? 4e9 : 2e9);
  return d >= 512 ? pairs >= nlist : products >= (d <= 96 ? 1e9 : 8e9);
}

// Whether such a request over lists of halves or bytes, squared distances, can scan on the 16-bit instructions (scan_mm.hip):
// wherever the vectors are wide enough to repay the queries' splitting, and three pieces of 16 queries fit beside another
// workgroup's in LDS.  4x4x1 / 16-bit, us a request (queries of three pieces), 256 lists:
//  bytes, 128 queries x 32 probes, lists of 600: d 16 44 / 47, d 32 48 / 46, d 64 58 / 48, d 128 71 / 56, d 320
//    128 / 81, d 640 192 / 144; 256 x 32, lists of 1,500: d 16 58 / 63, d 32 65 / 64, d 128 115 / 79, d 640 372 /
//    264; 64 x 8, of 1,500: d 64 47 / 46, d 128 56 / 53, d 640 173 / 154
//  halves, 128 x 32, lists of 600: d 16 46 / 45, d 32 50 / 45, d 128 74 / 58, d 320 128 / 86, d 640 196 / 154;
//    256 x 32, of 1,500: d 16 60 / 59, d 128 114 / 84, d 640 434 / 370; 64 x 8, of 1,500: d 64 49 / 50, d 128 54 /
//    55, d 640 124 / 124
inline bool narrow_scan_fits(const Dev &D) {
  return D.metric == 0 && D.pq_m == 0 && D.storage != 0 && D.d >= (D.storage == 2 ? 64 : 32) && D.d <= 640;
}
// ... and whether it should.  Nearly always; but an instruction takes 16 queries whether they are there or not, and an item's
// queries are split anew, which a tile of few repays only if its loads keep coming, and where a vector is a power of two of
// 16-byte chunks, the groups that wavefronts read side by side lie a power of two apart and memory answers more slowly.
// There it goes by the pairs to a list and by what the lists come to (past some 300 MB they come from HBM); hot lists,
// whose tiles are full, make little difference to where the line lies.  4x4x1 / 16-bit, us a request, over 1,900 requests of
// 64 to 256 queries x 4 to 64 probes over 64 to 4,096 lists: bytes, 1,024 lists of 4,000 x 256, 2 pairs to a list 224 / 269, 4
// 285 / 323, 6 340 / 348; of 1,000 x 128 4 pairs 0.93 to 0.95 of the time, 8 0.78 to 0.87; halves, 1,024 of 4,000 x 256, 4
// pairs 386 / 413, 8 428 / 449, 256 of 1,500 x 512, 8 pairs 162 / 147, 512 of 600 x 256, 4 pairs 99 / 90, x 32 55 / 58.  Bytes
// of 64 dimensions gain at any number of pairs where the lists are 60 MB and more (1,024 of 4,000, 2 pairs: 140 / 121; 512
// of 600: 57 / 60).  Other numbers of chunks: bytes, 1,024 of 2,000 x 192, 2 pairs 141 / 125, x 320 202 / 169, x 352 272 / 192, x
// 384 210 / 182; halves, 512 of 3,600 x 288, 4 pairs 272 / 247, x 352 328 / 294, x 400 337 / 311.
// Over 2,049 requests the rule is 0.3 % from the better of the two on average and at most 10 % behind (640 dimensions of
// bytes, 2 pairs: 192 / 211); always the 16-bit instructions are up to 20 % behind, never are up to 1.8 times as slow.
inline bool narrow_scan_pays(const Dev &D, int64_t pairs, double list_bytes) {
  const int64_t nlist = D.nlist;
  if (D.vchunks & (D.vchunks - 1)) return true;
  if (D.storage == 2) return pairs > 4 * nlist || (pairs > 2 * nlist && list_bytes < 300e6) || (D.d <= 64 && list_bytes >= 60e6);
  return pairs > 8 * nlist || (pairs == 8 * nlist && list_bytes < 500e6) ||
         (pairs >= 4 * nlist + (D.d < 128 ? 1 : 0) && list_bytes < 300e6);
}

// Whether a request over lists of floats with halves beside them reads those.  What speaks for them is bytes: the lists it meets, once
// each, and a fifth of what its pairs meet (squared distances: 16-bit instructions have the better of the arithmetic as well).
// What speaks against them is what is scored again, which goes with the dimensions and with k, in a few compute units when there are
// few queries.  Floats / halves, us a request of 1 to 256 queries: 1 M x 128 bytes in 1,024 lists, 32 probes, k 100, 8 queries 67 / 73, 32 112 /
// 94, 256 192 / 125; 10 M x 96 in 4,096, inner products, 128 x 64, k 10 618 / 360; 5 M x 768 in 8,192, 64 x 32 740 / 492; 20 M x
// 256 in 16,384, hot lists, 256 x 64 2,870 / 1,670; but 132,802 x 912 in 88, inner products, 200 x 8, k 128 215 / 451, and
// 964,127 x 356 in 667, one of them a fifth of it, 8 x 2, k 100 57 / 124.  Over 8,485 requests for squared distances (d 24 to 512, 64 to
// 16,384 lists, even ones and hot ones) the rule is 1.3 % behind the better of the two on average, and 1.33 times at worst, never would
// be 13 %; over 5,565 for inner products (d 24 to 1,024) 0.6 % and 1.25 times, and 7 %.  One to seven queries for squared distances stay
// with the floats, whose scan leaves off early and scores nothing again (up to 1.6 times as slow, 1.15 times as fast on average).
// What the rule cannot see is how much of a request lies within the halves' margin, which grows with the vectors' length beside
// their distances (1 M x 128 as above, k 100, vectors 0.3 apart about centres of length 11; 32 / 256 queries: 76 / 81 and 161 / 120;
// all of them 30 away from zero in every coordinate 72 / 115 and 202 / 149; queries 100 times as long 102 / 121 and 187 / 158).
// Where it is most of the request, 800 us and more, the floats take over: halves_may_tell(), rtams.hip.
inline bool halves_scan_pays(const Dev &D, int64_t nq, int64_t nprobe, int64_t k, int64_t avg_len, int64_t max_len) {
  const int64_t pairs = nq * nprobe;
  const double per = D.d * 4e-6, hot = (double)max_len * (nq < 10 ? (double)nq / 10.0 : 1.0);  // MB of a vector; a tenth of the queries meet the longest list
  const double lists = ((double)(pairs < D.nlist ? pairs : D.nlist) * (double)avg_len + hot) * per;
  const double again = (double)k * D.d * 1e-4;
  if (D.metric != 0) return lists >= 130.0 + 0.4 * D.d + 140.0 * again;
  return nq >= 8 && lists + 0.2 * (double)nq * ((double)(nprobe * avg_len) + (double)max_len / 10.0) * per >= 100.0 + 0.2 * D.d + 60.0 * again;
}

// Whether a scan of halves has tiles of 32 queries instead of 16: half the passes over a list that so many meet, and a workgroup
// less on a compute unit.  Whole requests, tiles of 16 / 32, us: even lists, 16 pairs to each 110 / 109 (1 M x 128), 97 / 92 (2 M x
// 32), 332 / 274 (400 k x 768; inner products 282 / 286), 32 pairs 130 / 119, 118 / 103, 374 / 326, 64 pairs 367 / 263; but 8 pairs
// 115 / 116, 89 / 85, 244 / 254.  One hot list: the pairs that make a second tile of 16 are its own, and what it costs is paid by
// all others; by squared distances, 256 queries, 20 M x 256 in 16,384 lists of a Zipf law 1,809 / 1,658, 20 M x 96 in 4,096 1,029 / 942,
// 6 M x 256 in 1,024 980 / 851, where the list meets 24 queries or fewer 1.01 times as long (up to 1.10); but where the others are short,
// 12 M and 6 M x 256 in 16,384 lists, 1,093 / 1,179 and 663 / 704; wide, 6 M x 768 in 8,192, 2,514 / 2,591; or by inner
// products 12 M x 256 in 16,384 1,626 / 2,166, 6 M x 768 2,847 / 2,924.
inline bool wide_half_tiles_pay(const Dev &D, int64_t nq, int64_t nprobe, int64_t ntotal, int64_t longest) {
  if (nq * nprobe >= 16 * (int64_t)D.nlist) return true;
  return D.metric == 0 && D.d <= 256 && ntotal >= 1024 * (int64_t)D.nlist && nq * longest >= 24 * ntotal;
}

inline ScanShape scan_shape(const Dev &D, int item_budget) {
  ScanShape sh{};
  sh.mm = (D.scan_mfma != 0 || D.scan_halves != 0) && D.pq_m == 0;
  // room for an uneven split of the items over the XCDs
  const int items = item_budget + item_budget / 2;
  if (!sh.mm) {
    const size_t per_wave = (size_t)kScanTileQueries * D.d * sizeof(float);
    int waves = kScanWaves;  // as many (4, 2, 1) as fit their query tiles into 64 KiB of LDS
    while (waves > 1 && per_wave * waves > 65536) waves /= 2;
    sh.tile_q = kScanTileQueries;
    sh.seg_base = D.scan_single ? 1 : 2;
    sh.min_choice = 0;
    sh.items_per_wg = waves;
    sh.threads = waves * kWave;
    sh.lds = per_wave * waves;
    sh.grid = ((items + waves - 1) / waves + (int)kXcds - 1) / (int)kXcds * (int)kXcds;
    return sh;
  }
  if (D.scan_halves) {  // a query's halves and 16 bytes that spread the rows over the banks, its words, and what its scores are made of
    const size_t row = (size_t)half_row_units(D) * 16 + 16 + kHalfQueryWords * 4;
    const size_t rest = kMmWaves * (kHalfStageBytes + kHalfPlaces * 4) + kHalfConsts * kMmTileMax * 4, ring = kMmWaves * kHalfRing * kHalfStep;
    sh.tile_q = D.scan_halves == 2 ? 32 : 16;
    sh.seg_base = 2;
    sh.min_choice = D.scan_min_choice >= 0 ? D.scan_min_choice : D.d >= 512 ? 1 : 2;
    sh.items_per_wg = 1;
    sh.threads = kMmWaves * kWave;
    sh.lds = row * sh.tile_q + rest + ring;
    sh.grid = (items + (int)kXcds - 1) / (int)kXcds * (int)kXcds;
    return sh;
  }
  // a query of the tile: coordinates, one float4 of padding, its words (or its three pieces and its words)
  const bool narrow = scans_narrow(D);
  const size_t row = (narrow ? (size_t)3 * narrow_row_bytes(D) : (size_t)(D.d + 4) * sizeof(float)) + kMmQueryWords * 4;
  const size_t stage = kMmWaves * kMmStageBytes;
  int rows = kMmTileMax;
  // two workgroups should fit a CU side by side; a tile is never below 8 queries unless LDS cannot hold that
  while (rows > (narrow ? 16 : 8) && row * rows + stage > 64 * 1024) rows /= 2;
  while (rows > 4 && row * rows + stage > kMmLdsMax) rows /= 2;
  sh.tile_q = rows;
  sh.seg_base = 2;
  sh.min_choice = 2;  // at least 8 groups to an item, two for every wavefront (measured: 4 and 16 are slower)
  if (D.scan_min_choice >= 0) sh.min_choice = D.scan_min_choice;
  sh.items_per_wg = 1;
  sh.threads = kMmWaves * kWave;
  sh.lds = row * rows + stage;
  sh.grid = (items + (int)kXcds - 1) / (int)kXcds * (int)kXcds;
  return sh;
}

// Workgroup of the planning kernel (k_group).  Two of them fit a CU side by side, so that a request
// of as many queries as the chip has CUs, with its two extra workgroups, still starts all at once
// (with 1024 threads the last two waited for the first to finish: 17 us at 256 queries).
constexpr int kGroupThreads = 512;

}  // namespace rtams
