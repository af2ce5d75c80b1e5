// The pruning bound of a query, set by one workgroup.
#pragma once
#include "search_common.h"

namespace rtams {

// ------------------------------------------------------------- pruning bound
constexpr int kSampleMax = 4096;  // candidates the bound of a query is taken from, at most
#ifndef RTAMS_SAMPLE_DIVISOR
#define RTAMS_SAMPLE_DIVISOR 4
#endif
constexpr int kSampleDivisor = RTAMS_SAMPLE_DIVISOR;
constexpr int kNoBoundBelow = 4096;  // candidates of a query up to which the scan keeps them all

// The scan writes nothing for a candidate that cannot be among the k best of
// its query: before it starts, every query gets a BOUND, the k-th best score
// of a sample of its candidates (the first few groups of its nearest probed
// lists, where most of its neighbours are).  The k-th best of any k or more
// candidates cannot be better than the final k-th best, so keeping what is not
// worse than the bound loses nothing.  One workgroup to a query, or several that
// share its sample (below): a wavefront per group of 64 vectors, lane = vector,
// scores to LDS, radix selection there.
// These workgroups run beside the one that groups the pairs (same launch): both
// need only the plan, and the scan needs both.
// What the sample needs of the nearest list, read ahead by the caller (every one of these is a round
// trip to memory, and read where they are used they would follow one another): the list, its
// length, its number of blocks, and where the table segment of this wavefront's first group starts.
struct NearestList {
  int list;
  uint32_t len, nblk;
  int32_t dir;
};

template <int METRIC, int ST>
__device__ uint32_t sample_scores(const Dev &D, int nprobe, int max_nprobe, int q, uint32_t want_groups,
                              const float *__restrict__ Q, const SearchScratch &S, const float4 *qv,
                              uint32_t *skey, uint32_t *gkey, uint32_t part, uint32_t parts, const NearestList &first) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const uint32_t mine = (uint32_t)(tid / kWave) * parts + part, step = blockDim.x / kWave * parts;
  const int d4 = D.vchunks;  // 16-byte chunks of a stored vector
  constexpr int kPieces = pieces_of(ST);  // float4s of the query that go with a chunk
  const uint32_t gpb = (uint32_t)D.groups_per_block;
  const size_t group_stride = (size_t)d4 * kWave;
  // the sample is the first want_groups groups of the probed lists taken in order, nearest first
  uint32_t g_first = 0;  // groups of the lists before list p
  for (int p = 0; p < nprobe && g_first < want_groups; ++p) {  // uniform over the workgroup
    const size_t o = (size_t)q * max_nprobe + p;
    const int list = p == 0 ? first.list : S.probe_list[o];
    const uint32_t len = p == 0 ? first.len : S.probe_len[o];
    uint32_t groups = (len + kWave - 1) / kWave;
    const uint32_t have = (p == 0 ? first.nblk : D.nblk[list]) * gpb;  // never index the block table past the chain
    if (groups > have) groups = have;
    if (groups > want_groups - g_first) groups = want_groups - g_first;
    for (uint32_t g = mine; g < groups; g += step) {
      const uint32_t b = p == 0 && g == mine ? (uint32_t)*table_entry_at(D, first.dir, g / gpb)
                                                       : (uint32_t)*table_entry(D, list, g / gpb);
      const float4 *__restrict__ x = block_vecs(D, b) + (size_t)(g % gpb) * group_stride + lane;
      float acc = 0.f;
      int c = 0;
      if (METRIC == 1 && D.scan_mfma) {
        // inner products on the matrix cores, exactly as the scan computes them (same
        // instruction, same order of the coordinates), so that a candidate's score here and there is
        // the same bits: every lane offers the one query, component l % 4 of the result is the score
        // of the lane's own vector
        MfmaAcc m = {0.f, 0.f, 0.f, 0.f};
        if (ST == 0)
          for (; c + 16 <= d4; c += 16) {
            float4 v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = x[(size_t)(c + u) * kWave];
#pragma unroll
            for (int u = 0; u < 16; ++u) mfma_chunk(m, v[u], qv[c + u]);
          }
        for (; c + 8 <= d4; c += 8) {
          float4 v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = x[(size_t)(c + u) * kWave];
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int s = 0; s < kPieces; ++s) mfma_chunk(m, chunk_piece<ST>(v[u], s), qv[(c + u) * kPieces + s]);
        }
        for (; c < d4; ++c) {
          const float4 v = x[(size_t)c * kWave];
#pragma unroll
          for (int s = 0; s < kPieces; ++s) mfma_chunk(m, chunk_piece<ST>(v, s), qv[c * kPieces + s]);
        }
        const int r = lane & 3;
        acc = r == 0 ? m[0] : r == 1 ? m[1] : r == 2 ? m[2] : m[3];
      }
      // loads of 1 KiB in flight per wavefront: sixteen, then eight, then one at a time (the workgroup
      // is alone on its CU and a group is a chain of such round trips)
      if (ST == 0) {
        for (; c + 16 <= d4; c += 16) {
          float4 v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) v[u] = x[(size_t)(c + u) * kWave];
#pragma unroll
          for (int u = 0; u < 16; ++u) accumulate<METRIC>(acc, v[u], qv[c + u]);
        }
      }
      for (; c + 8 <= d4; c += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[(size_t)(c + u) * kWave];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int s = 0; s < kPieces; ++s) accumulate<METRIC>(acc, chunk_piece<ST>(v[u], s), qv[(c + u) * kPieces + s]);
      }
      for (; c < d4; ++c) {
        const float4 v = x[(size_t)c * kWave];
#pragma unroll
        for (int s = 0; s < kPieces; ++s) accumulate<METRIC>(acc, chunk_piece<ST>(v, s), qv[c * kPieces + s]);
      }
      const uint32_t v = g * kWave + lane;
      const uint32_t key = v < len ? key_of_float((METRIC == 0 ? acc : -acc) + 0.0f) : 0xFFFFFFFFu;
      const size_t at = (size_t)(g_first + g) * kWave + lane;
      if (gkey) __hip_atomic_store(&gkey[at], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // uniform
      else skey[at] = key;
    }
    g_first += groups;
  }
  return g_first;  // groups the lists did not have stay at the worst key (set by the caller)
}

// The same sample from the halves beside the lists: half the bytes, and a compute unit reads no more than so many at once.  A score is
// of the query against what the halves hold; what they leave out goes into the bound where it is used (halves_bound_key),
// for inner products but what depends on the vector, `over` times its length, which is added here: the score is then no less than
// the vector's own.
template <int METRIC>
__device__ uint32_t sample_scores_halves(const Dev &D, int nprobe, int max_nprobe, int q, uint32_t want_groups, const SearchScratch &S,
                                         const float4 *qv, float over, uint32_t *skey, uint32_t *gkey, uint32_t part, uint32_t parts,
                                         const NearestList &first) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), hc = D.hchunks;
  const uint32_t mine = (uint32_t)(tid / kWave) * parts + part, step = blockDim.x / kWave * parts;
  const uint32_t gpb = (uint32_t)D.groups_per_block;
  const float ixs = 1.f / halves_scale(D);
  const int sub = lane & 3, of16 = lane >> 2, quads = (hc + 3) / 4;  // the lane's chunk of four, and its vector of each 16
  uint32_t g_first = 0;  // groups of the lists before list p
  for (int p = 0; p < nprobe && g_first < want_groups; ++p) {  // uniform over the workgroup
    const size_t o = (size_t)q * max_nprobe + p;
    const int list = p == 0 ? first.list : S.probe_list[o];
    const uint32_t len = p == 0 ? first.len : S.probe_len[o];
    uint32_t groups = (len + kWave - 1) / kWave;
    const uint32_t have = (p == 0 ? first.nblk : D.nblk[list]) * gpb;  // never index the block table past the chain
    if (groups > have) groups = have;
    if (groups > want_groups - g_first) groups = want_groups - g_first;
    for (uint32_t g = mine; g < groups; g += step) {
      const uint32_t b = p == 0 && g == mine ? (uint32_t)*table_entry_at(D, first.dir, g / gpb) : (uint32_t)*table_entry(D, list, g / gpb);
      const char *__restrict__ x = block_halves(D, b) + (size_t)(g % gpb) * ((size_t)hc * (kWave * 16));
      float acc[4] = {0.f, 0.f, 0.f, 0.f}, nrm[4] = {0.f, 0.f, 0.f, 0.f};
      auto load = [&](u32x4 *v, int quad) {  // the lane's chunk of vector 16 b + of16
        const int width = min(hc - 4 * quad, 4), s = min(sub, width - 1);
#pragma unroll
        for (int b4 = 0; b4 < 4; ++b4) v[b4] = *reinterpret_cast<const u32x4 *>(x + (size_t)quad * (kWave * 64) + ((16 * b4 + of16) * width + s) * 16);
      };
      auto use = [&](const u32x4 *v, int quad) {
        const bool on = 4 * quad + sub < hc;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float4 y = qv[on ? 8 * quad + 2 * sub + s : 0];
          if (!on) y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int b4 = 0; b4 < 4; ++b4) {
            const uint32_t w0 = on ? v[b4][2 * s] : 0u, w1 = on ? v[b4][2 * s + 1] : 0u;
            const Half2 a = __builtin_bit_cast(Half2, w0), e = __builtin_bit_cast(Half2, w1);
            accumulate<METRIC>(acc[b4], make_float4((float)a.x * ixs, (float)a.y * ixs, (float)e.x * ixs, (float)e.y * ixs), y);
            if (METRIC == 1) nrm[b4] = __builtin_amdgcn_fdot2(e, e, __builtin_amdgcn_fdot2(a, a, nrm[b4], false), false);
          }
        }
      };
      int quad = 0;
      for (; quad + 3 <= quads; quad += 3) {  // 12 loads of 1 KiB in flight
        u32x4 v[3][4];
#pragma unroll
        for (int u = 0; u < 3; ++u) load(v[u], quad + u);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          use(v[u], quad + u);
          __builtin_amdgcn_sched_barrier(0);  // one step's widened values at a time
        }
      }
      for (; quad + 2 <= quads; quad += 2) {
        u32x4 v[2][4];
        load(v[0], quad);
        load(v[1], quad + 1);
        use(v[0], quad);
        use(v[1], quad + 1);
      }
      if (quad < quads) {
        u32x4 v[4];
        load(v, quad);
        use(v, quad);
      }
      // the four lanes of a vector have its sum between them; lane s of the four goes on with vector 16 s + of16
      float mine = 0.f, mine_n = 0.f;
#pragma unroll
      for (int b4 = 0; b4 < 4; ++b4) {
        float a = acc[b4] + quad_xor<1>(acc[b4]), n = nrm[b4];
        a += quad_xor<2>(a);
        if (METRIC == 1) { n += quad_xor<1>(n); n += quad_xor<2>(n); }
        mine = sub == b4 ? a : mine;
        mine_n = sub == b4 ? n : mine_n;
      }
      const uint32_t in_group = 16u * (uint32_t)sub + (uint32_t)of16, v = g * kWave + in_group;
      const float sc = METRIC == 0 ? mine : fmaf(over, sqrtf(mine_n) * ixs, -mine);
      const uint32_t key = v < len && fabsf(sc) < __builtin_inff() ? key_of_float(sc + 0.0f) : 0xFFFFFFFFu;
      const size_t at = (size_t)(g_first + g) * kWave + in_group;
      if (gkey) __hip_atomic_store(&gkey[at], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // uniform
      else skey[at] = key;
    }
    g_first += groups;
  }
  return g_first;
}

// The same sample over product-quantiser codes: a vector's score is the sum, in the order of the
// sub-spaces, of the entries of the query's table (in LDS) that its codes name.  What a wavefront needs of its group of
// the nearest list is read ahead by the caller, while the table is made: five trips to memory, one behind the other.
constexpr int kPqAhead = 4;  // words of codes of a vector
struct PqNearest {
  int list;
  uint32_t len, nblk;
  uint32_t code[kPqAhead];
};
__device__ __forceinline__ const uint32_t *pq_group(const Dev &D, int list, uint32_t g) {
  const uint32_t gpb = (uint32_t)D.groups_per_block, b = (uint32_t)*table_entry(D, list, g / gpb);
  return block_codes(D, b) + (size_t)(g % gpb) * (D.pq_m / 4) * kWave + (threadIdx.x & (kWave - 1));
}
__device__ __forceinline__ PqNearest pq_nearest(const Dev &D, int max_nprobe, int q, const SearchScratch &S) {
  const size_t o = (size_t)q * max_nprobe;
  PqNearest first{S.probe_list[o], S.probe_len[o], 0u, {}};
  first.nblk = D.nblk[first.list];
  const uint32_t g = threadIdx.x / kWave;
  if (g < min((first.len + kWave - 1) / kWave, first.nblk * (uint32_t)D.groups_per_block)) {  // uniform over the wavefront
    const uint32_t *x = pq_group(D, first.list, g);
#pragma unroll
    for (int c = 0; c < kPqAhead; ++c) first.code[c] = x[(size_t)min(c, D.pq_m / 4 - 1) * kWave];
  }
  return first;
}
__device__ void pq_sample_scores(const Dev &D, int nprobe, int max_nprobe, int q, uint32_t want_groups,
                                 const SearchScratch &S, const float *lut, const PqNearest &first, uint32_t *skey) {
  const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int words = D.pq_m / 4;
  uint32_t g_first = 0;
  for (int p = 0; p < nprobe && g_first < want_groups; ++p) {  // uniform over the workgroup
    const size_t o = (size_t)q * max_nprobe + p;
    const int list = p == 0 ? first.list : S.probe_list[o];
    const uint32_t len = p == 0 ? first.len : S.probe_len[o];
    uint32_t groups = (len + kWave - 1) / kWave;
    const uint32_t have = (p == 0 ? first.nblk : D.nblk[list]) * (uint32_t)D.groups_per_block;  // never index the block table past the chain
    if (groups > have) groups = have;
    if (groups > want_groups - g_first) groups = want_groups - g_first;
    for (uint32_t g = wave; g < groups; g += blockDim.x / kWave) {
      const bool ahead = p == 0 && g == wave;  // uniform over the wavefront
      const uint32_t *__restrict__ x = ahead && words <= kPqAhead ? nullptr : pq_group(D, list, g);
      float acc = 0.f;
      for (int c0 = 0; c0 < words; c0 += kPqAhead) {
        uint32_t w[kPqAhead];
#pragma unroll
        for (int c = 0; c < kPqAhead; ++c) w[c] = ahead && c0 == 0 ? first.code[c] : x[(size_t)min(c0 + c, words - 1) * kWave];
#pragma unroll
        for (int c = 0; c < kPqAhead; ++c)
          if (c0 + c < words) {
            const float *t = lut + (size_t)(c0 + c) * 4 * 256;
            acc += t[w[c] & 255u];
            acc += t[256 + ((w[c] >> 8) & 255u)];
            acc += t[512 + ((w[c] >> 16) & 255u)];
            acc += t[768 + (w[c] >> 24)];
          }
      }
      const uint32_t v = g * kWave + lane;
      skey[(size_t)(g_first + g) * kWave + lane] =
          v < len ? key_of_float((D.metric == 0 ? acc : -acc) + 0.0f) : 0xFFFFFFFFu;
    }
    g_first += groups;
  }
}

// LDS of a bound: the query (d <= 2048; none where a table is) and the keys of the sample.  The caller owns it, so that a
// kernel whose workgroups do different jobs can use the same bytes for each.
constexpr size_t kBoundLdsBytes = 512 * sizeof(float4) + kSampleMax * sizeof(uint32_t);
constexpr size_t kPqBoundLdsBytes = kSampleMax * sizeof(uint32_t);

// A request of few queries leaves compute units idle while one of them reads a sample of wide vectors or of a long list:
// three or kSampleParts workgroups read it then (part of parts), leave the keys in the row of the query's approximate scores,
// which nobody needs any more, and the last one goes on.  One compute unit reads 40 to 60 GB/s however much it asks for at
// once; this launch, with one workgroup to a query and with several (us): 64 queries over lists of 610 x 768 floats, samples
// of 1,536 chunks of 1 KiB, 34.8 / 20.9; 128 queries over lists of 2,441 x 96, 192 to 1,000 chunks, 51.4 / 27.1.
// Whole requests, shared against not, 32 probes: samples of eight groups 0.93 to 0.99 of the time from 512 chunks up to 64
// queries and 0.99 to 1.01 at 120 to 160, from 288 to 400 chunks 0.98 to 1.01; of a quarter of lists of 3,600 x 96, 336
// chunks, 0.96 to 0.98 at 120 to 160; eight groups of 256 chunks and fewer 1.00 to 1.04, so such a sample is left to one:
// the hand-over between the workgroups is a microsecond.  Two workgroups to a query (168 queries and more) are 1 to 1.5 %
// behind one.
constexpr int kSampleParts = 4;
constexpr uint32_t kSplitChunks = 260;

// A query's halves and what goes with them (half_query_row), by one wavefront, and `over` of its sample.  (Workgroups that share the
// sample all write the row; should they find halves_are_floats different, either is right.)
__device__ inline void make_half_query(const Dev &D, const SearchScratch &S, int q, const float *__restrict__ Q, float *over_out) {
  const int lane = threadIdx.x & (kWave - 1);
  const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
  double nsq = 0.0;
  for (int c = lane; c < D.d4; c += kWave) {
    const float4 v = y[c];
    nsq += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
  }
  for (int o = kWave / 2; o > 0; o >>= 1) nsq += __shfl_xor(nsq, o);
  const float scale = half_query_scale(nsq), inv = 1.f / scale;
  u32x4 *row = half_query_row(D, S, (uint32_t)q);
  double hsq = 0.0, rsq = 0.0;  // |q'|^2 and |q - q'|^2
  for (int c = lane; c < (int)half_row_units(D); c += kWave) {
    uint2 h[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const bool on = 2 * c + p < D.d4;
      float4 v = y[on ? 2 * c + p : 0];
      if (!on) v = make_float4(0.f, 0.f, 0.f, 0.f);
      bool exact = true;
      h[p] = pack_four_halves(v, scale, exact);
      const float4 b = chunk_piece<1>(make_float4(__uint_as_float(h[p].x), __uint_as_float(h[p].y), 0.f, 0.f), 0);
      auto add = [&](float have, float want) {
        const double t = (double)have * (double)inv, r = (double)want - t;
        hsq += t * t;
        rsq += r * r;
      };
      add(b.x, v.x); add(b.y, v.y); add(b.z, v.z); add(b.w, v.w);
    }
    row[c] = u32x4{h[0].x, h[0].y, h[1].x, h[1].y};
  }
  for (int o = kWave / 2; o > 0; o >>= 1) { hsq += __shfl_xor(hsq, o); rsq += __shfl_xor(rsq, o); }
  if (lane == 0) {
    const float norm = (float)__builtin_sqrt(nsq > hsq ? nsq : hsq) * 1.00001f, left = (float)__builtin_sqrt(rsq) * 1.00001f;
    const bool exact = halves_are_floats(D);
    *reinterpret_cast<float4 *>(row + half_row_units(D)) = make_float4(exact ? -inv : inv, (float)hsq, norm, left);
    *over_out = halves_over(norm, exact, D.d);
  }
}

// HALVES: the request reads the halves beside the lists
template <bool PQ, bool HALVES>
__device__ void sample_bound(const Dev &D, int q, int nprobe, int max_nprobe, int k, const float *__restrict__ Q,
                             const SearchScratch &S, unsigned char *lds, uint32_t part, uint32_t parts,
                             const float *lut = nullptr, const PqNearest &nearest = PqNearest{}) {
  float4 *qv = reinterpret_cast<float4 *>(lds);
  uint32_t *skey = reinterpret_cast<uint32_t *>(lds + (PQ ? 0 : 512 * sizeof(float4)));
  __shared__ __attribute__((aligned(8))) uint32_t hist[kSelectLdsWords];
  __shared__ uint32_t bc[4];
  const int tid = threadIdx.x;
  // what decides how the workgroup goes on, all on its way at once
  const size_t o0 = (size_t)q * max_nprobe;
  const uint32_t qtotal = S.qtotal[q];
  NearestList first{PQ ? 0 : S.probe_list[o0], PQ ? nearest.len : S.probe_len[o0], 0u, 0};
  // |q|^2 for the norm form of the squared distance (the first wavefront computes it, in double)
  constexpr bool halves = HALVES;
  const bool norm_form = !PQ && !halves && uses_norm_form(D);
  __shared__ float s_qn;
  __shared__ float s_over;
  if (halves && tid < kWave) make_half_query(D, S, q, Q, &s_over);
  if (norm_form && tid < kWave) {
    double a = 0.0;
    for (int c = tid; c < D.d; c += kWave) {
      const double v = (double)Q[(size_t)q * D.d + c];
      a = __builtin_fma(v, v, a);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_xor(a, o);
    if (tid == 0) { s_qn = (float)a; S.qnorm[q] = (float)a; }
  }
  // A query with no more candidates than the selection holds in LDS at once needs no bound.  For
  // inner products neither does one whose records cost less than a sample would: the sample is 512
  // vectors or more, a record is 8 bytes (short lists, wide vectors).  Requests of 1 to 256 queries without a bound against
  // with one, up to 32 d candidates: d 256 0.93 to 1.12 of the time, d 384 0.92 to 1.16, d 768 0.56 to 1.08, d 1024 0.52 to
  // 1.14, the large ones where long lists meet few of the candidates.  (For L2 the bound also lets the scan stop early,
  // which is worth the sample.)
  const uint32_t no_bound_below =
      D.metric == 0 || halves ? (uint32_t)kNoBoundBelow : max((uint32_t)kNoBoundBelow, 32u * (uint32_t)D.d);
  auto keep_everything = [&]() {
    if (tid == 0 && part == 0) {
      S.bound[q] = 0xFFFFFFFFu;
      if (halves) rec_words_clear(S, (uint32_t)q);
      else *rec_count(S, (uint32_t)q) = 0u;
    }
  };
  if (qtotal <= no_bound_below) {  // uniform over the workgroup
    keep_everything();
    return;
  }
  // sample size: 4 k, at least 512 and at least a fraction of the nearest list (the longer that
  // list, the more candidates a given score admits), at most kSampleMax and, but for the 512, at most
  // 1 MiB of vectors (with the rounding below a third more; a hot list of wide vectors would hold up the scan), in whole groups
  const uint32_t chunks = halves ? (uint32_t)D.hchunks : (uint32_t)D.vchunks;  // 16 bytes each, of a vector of the sample
  uint32_t cap = PQ ? (uint32_t)kSampleMax : ((1u << 20) / (chunks * 16u)) & ~(uint32_t)(kWave - 1);
  // ... and for squared distances what k needs: a sample of fewer than k vectors is no bound at all, every candidate is then
  // kept and scored again (176 queries x 45 probes over lists of up to 144,000 x 1,036 floats, k 703: 19.0 ms a request without
  // a bound, 14.9 with; 64 queries x 32 over lists of 1,000 x 1,536 bytes, k 1,000: 0.13 of the time; inner products, which
  // score nothing again, were up to 1.44 times as slow with so large a sample)
  const uint32_t least = max(512u, (uint32_t)k + (uint32_t)k / 4u);
  cap = min(max(cap, D.metric == 0 ? (least + kWave - 1) & ~(uint32_t)(kWave - 1) : 512u), (uint32_t)kSampleMax);
  uint32_t want = (uint32_t)k * 4u;
  const uint32_t share = first.len / (uint32_t)kSampleDivisor;
  want = want < share ? share : want;
  want = want < 512u ? 512u : (want > cap ? cap : want);
  uint32_t want_groups = (want + kWave - 1) / kWave;
  if (!PQ) {
    if (parts > 1 && (want_groups * chunks < kSplitChunks || want_groups * kWave > (uint32_t)D.nlist)) {
      if (part) return;  // uniform, and the same for all workgroups of the query
      parts = 1;
    }
    // A sample is the nearest number of whole turns of the wavefronts that read it, a group to each, if it is more than one
    // turn (256 queries over lists of 2,441 x 96, ten groups to one workgroup: the last two were a turn of their own; 128
    // queries, three workgroups, up to 35 groups: this launch 27 us with 24 and 33 with 35), but no fewer than a quarter more
    // than k as far as the cap goes (256 queries, k 600, lists of 1,560 x 400: 557 us a request with eight groups, which are
    // no bound, 455 with ten).  Up to one turn is not rounded: eight groups, sixteen for two workgroups, made 305 us of 200
    // queries over lists of 600 x 384 that take 279 with eight and one.  And that quarter more than k is enough for several
    // (64 queries over lists of 364 x 300, k 200: 159 us with eight groups, 165 with 4 k's thirteen; k 500: 234 with eight,
    // 206 with ten or thirteen).
    const uint32_t turn = blockDim.x / kWave * parts;
    if (parts > 1) want_groups = min(want_groups, (max(least, share) + kWave - 1) / kWave);
    if (want_groups > turn) {
      const uint32_t whole = (want_groups + turn / 2) / turn * turn;
      want_groups = min(max(whole, min(want_groups, (least + kWave - 1) / kWave)), (uint32_t)kSampleMax / kWave);
      if (parts > 1) want_groups = min(want_groups, (uint32_t)D.nlist / kWave);
    }
    // a sample of fewer than k vectors (lists end inside a group) is no bound and need not be read
    if ((uint32_t)k * 2u > want_groups * kWave) {  // uniform
      uint32_t groups = 0, vectors = 0;
      for (int p = 0; p < nprobe && groups < want_groups; ++p) {
        const uint32_t len = S.probe_len[o0 + p], take = min((len + kWave - 1) / kWave, want_groups - groups);
        groups += take;
        vectors += min(len, take * kWave);
      }
      if (vectors < (uint32_t)k) {
        keep_everything();
        return;
      }
    }
    // on their way while the query and the keys are set up
    first.nblk = D.nblk[first.list];
    first.dir = table_dir(D, first.list, ((uint32_t)(tid / kWave) * parts + part) / (uint32_t)D.groups_per_block);
  }
  if (!PQ)
    for (int c = tid; c < (HALVES ? 2 * D.hchunks : D.d4); c += (int)blockDim.x)
      qv[c] = !HALVES || c < D.d4 ? reinterpret_cast<const float4 *>(Q + (size_t)q * D.d)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i = tid; i < (int)(want_groups * kWave); i += (int)blockDim.x) skey[i] = 0xFFFFFFFFu;
  __syncthreads();
  if (PQ) {
    pq_sample_scores(D, nprobe, max_nprobe, q, want_groups, S, lut, nearest, skey);
  } else {
    uint32_t *gkey = parts > 1 ? reinterpret_cast<uint32_t *>(S.approx) + (size_t)q * D.nlist : nullptr;
    uint32_t groups;
    if (HALVES) {  // (of a request that reads halves)
      groups = D.metric == 0 ? sample_scores_halves<0>(D, nprobe, max_nprobe, q, want_groups, S, qv, s_over, skey, gkey, part, parts, first)
                             : sample_scores_halves<1>(D, nprobe, max_nprobe, q, want_groups, S, qv, s_over, skey, gkey, part, parts, first);
    } else if (D.metric == 0) {
      if (D.storage == 1) groups = sample_scores<0, 1>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
      else if (D.storage == 2) groups = sample_scores<0, 2>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
      else groups = sample_scores<0, 0>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
    } else {
      if (D.storage == 1) groups = sample_scores<1, 1>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
      else if (D.storage == 2) groups = sample_scores<1, 2>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
      else groups = sample_scores<1, 0>(D, nprobe, max_nprobe, q, want_groups, Q, S, qv, skey, gkey, part, parts, first);
    }
    if (parts > 1) {  // uniform
      __shared__ uint32_t s_last;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's keys are out ...
      __syncthreads();                                  // ... and so are everybody's before the workgroup counts itself off
      if (tid == 0) {
        s_last = atomicAdd(&S.done_count[q], 1u) + 1u == parts;
        if (s_last) S.done_count[q] = 0u;  // (a small request expects it at zero)
      }
      __syncthreads();
      if (!s_last) return;  // uniform: the last one goes on
      for (uint32_t i = (uint32_t)tid; i < groups * kWave; i += blockDim.x)
        skey[i] = __hip_atomic_load(&gkey[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  // k-th smallest key of the sample; with fewer than k candidates in it, it is the worst key
  // and everything is kept
  uint32_t bound = 0xFFFFFFFFu;
  if ((uint32_t)k <= want_groups * kWave) {
    const SelectResult r = wg_radix_select<32>(
        (int)(want_groups * kWave), (uint32_t)k, [&](int i, uint64_t &kv) { kv = skey[i]; return true; }, hist, bc,
        (uint32_t)(k + k / 16));
    bound = (uint32_t)r.T;  // the k-th smallest key, or an upper bound of it that admits the same candidates
  }
  if (tid == 0) {
    // the sample's scores are direct-form ones; the scan may compare norm-form scores with the bound
    if (norm_form) bound = loosened_key(bound, norm_form_slack(D.d), s_qn);
    S.bound[q] = bound;
    if (halves) rec_words_clear(S, (uint32_t)q);
    else *rec_count(S, (uint32_t)q) = 0u;
  }
}

}  // namespace rtams
