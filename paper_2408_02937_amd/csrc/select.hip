// Top-k selection: the k best of every query's survivor records, by (score, id).
#include "search_common.h"

namespace rtams {

// ------------------------------------------------------------ top-k selection
// One workgroup per query takes the k best of the query's survivor records
// (what the scan appended for it) by (score, id): exact selection with the id
// tie-break, then a sort of the winners.  The records
// number a few hundred as a rule and are worked on in LDS; a list longer than
// LDS holds (massive ties) is selected from in place.
constexpr int kSurvivorCap = 4096;

constexpr int kTieCap = 1024;  // candidates tied at the k-th score that are told apart in LDS

struct SelectShared {
  __attribute__((aligned(8))) uint32_t hist[kSelectLdsWords];
  uint32_t bc[4];
  uint32_t cnt[2];
  uint64_t k1[kMaxK];
  uint64_t k2[kMaxK];
  uint32_t pay[kMaxK];
  uint64_t tie_id[kTieCap];
  uint32_t tie_item[kTieCap];
};

// Exact top-k among `count` items given by key(j) (32-bit score key) and
// item(j) (the candidate's place in the pool, for the id lookup).  Leaves the winners sorted in
// sh.k1 (score key), sh.k2 (id key), sh.pay (place in the pool); returns how
// many.  Candidates tied at the k-th score are told apart by id: their ids are
// fetched once and ranked in LDS (with byte-valued data such ties are the rule,
// a handful per query); only more ties than kTieCap go through a radix
// selection over the ids.
template <typename KeyFn, typename ItemFn, typename IdFn>
__device__ __forceinline__ int select_topk(int count, int k, KeyFn key, ItemFn item, IdFn id_of, SelectShared &sh) {
  auto key_of_id = [](int64_t id) -> uint64_t { return (uint64_t)id ^ 0x8000000000000000ull; };
  const int kk = k < count ? k : count;
  SelectResult r1{~0ull, 0, 0}, r2{~0ull, 0, 0};
  // What is taken is sorted by (score, id) anyway: a threshold that admits a few more than k does, and settles most ties
  // at the k-th score on the way.  (One query over 1 M x 128 bytes, 2,300 records, k 100: the whole selection 11.8 us before,
  // 10.2 with this, the ids fetched together and the branch taken out of the sort; room for 64 more instead of 16 cost
  // the sort what the passes saved, 13.5.)  No more than those, and they are all taken without a threshold (some 20 records, k 16:
  // 5.9 us with the passes over them, 4.4 without).
  const uint32_t room = (uint32_t)min(k + 16, kMaxK);
  const bool all = count <= (int)room;
  if (!all)
    r1 = wg_radix_select<32>(count, (uint32_t)k, [&](int j, uint64_t &kv) { kv = key(j); return true; },
                             sh.hist, sh.bc, room);
  const bool few = !all && (uint32_t)k - r1.need + r1.c_eq <= room;  // all that are not worse than T are taken
  const bool tie_break = !all && !few;  // more candidates tied at the k-th score than are sorted
  const bool in_lds = tie_break && r1.c_eq <= (uint32_t)kTieCap;
  if (tie_break && !in_lds)
    r2 = wg_radix_select<64>(count, r1.need,
                             [&](int j, uint64_t &kv) {
                               if (key(j) != (uint32_t)r1.T) return false;
                               kv = key_of_id(id_of(item(j)));
                               return true;
                             },
                             sh.hist, sh.bc);
  if (threadIdx.x == 0) sh.cnt[0] = sh.cnt[1] = 0;
  __syncthreads();
  // Winners and ties are collected by their places first, and the ids of all of them are fetched together: fetched where a
  // winner is found, an id was a trip to memory in every turn of this loop, and the ties' ids another behind it.
  for (int j = threadIdx.x; j < count; j += blockDim.x) {
    const uint32_t kv = key(j);
    bool take = all || kv < (uint32_t)r1.T || (kv == (uint32_t)r1.T && few);
    if (!take && kv == (uint32_t)r1.T) {
      if (in_lds) {
        sh.tie_item[atomicAdd(&sh.cnt[1], 1u)] = (uint32_t)item(j);
      } else {
        const uint64_t ik = key_of_id(id_of(item(j)));
        if (ik < r2.T) take = true;
        else if (ik == r2.T) take = atomicAdd(&sh.cnt[1], 1u) < r2.need;  // identical (score, id) pairs
      }
    }
    if (take) {
      const uint32_t p = atomicAdd(&sh.cnt[0], 1u);
      sh.k1[p] = kv; sh.pay[p] = (uint32_t)item(j);
    }
  }
  __syncthreads();
  {
    const int won = (int)sh.cnt[0], nt = in_lds ? (int)sh.cnt[1] : 0;
    for (int t = threadIdx.x; t < won + nt; t += blockDim.x) {
      const uint64_t ik = key_of_id(id_of(t < won ? (int)sh.pay[t] : (int)sh.tie_item[t - won]));
      if (t < won) sh.k2[t] = ik;
      else sh.tie_id[t - won] = ik;
    }
  }
  if (in_lds) {  // uniform over the workgroup
    const int nt = (int)sh.cnt[1];  // == r1.c_eq
    __syncthreads();
    for (int t = threadIdx.x; t < nt; t += blockDim.x) {
      const uint64_t mine = sh.tie_id[t];
      uint32_t rank = 0;
      for (int u = 0; u < nt; ++u) {
        const uint64_t other = sh.tie_id[u];
        rank += (other < mine || (other == mine && u < t)) ? 1u : 0u;
      }
      if (rank < r1.need) {
        const uint32_t p = atomicAdd(&sh.cnt[0], 1u);
        sh.k1[p] = (uint32_t)r1.T; sh.k2[p] = mine; sh.pay[p] = sh.tie_item[t];
      }
    }
    __syncthreads();
  }
  wg_sort<32>(all ? count : few ? (int)((uint32_t)k - r1.need + r1.c_eq) : kk, sh.k1, sh.k2, sh.pay);  // (of a few more than k the first k)
  return kk;
}

constexpr int kTopkThreads = 512;
constexpr int kSelectParts = 8;  // workgroups that share a query's finalists, at most
// ... where its records come to so many chunks of four coordinates.  Whole requests of 1 to 128 queries, d 32 to 1,536, one
// workgroup / several: below 5,000 several are 1.03 times as long on average (up to 1.07), at 7,000 to 11,000 1.01, at 13,000 to
// 16,000 0.95 by squared distances and 1.01 by inner products, at 25,000 to 28,000 0.92 and 0.98, above 50,000 0.88 and 0.96
// (one query by inner products 1.02: two turns of a chain each)
constexpr int64_t kSharedWork = 16384;

__device__ inline float score_of_key(uint32_t key, int metric) {
  const float x = __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
  return metric == 0 ? x : -x;
}

// ST: what flat lists keep (only the finalists' second scores depend on it: quantised lists take 0)
// (four wavefronts to a SIMD, or a compute unit takes one workgroup instead of two; measured with 129 registers and with
// 125: 256 queries over 1 M x 16 codes on four streams 74.5 / 73.7 us a request, float lists the same within noise)
// HALVES: the records are what the halves beside float lists can say (scan_halves.hip).  METRIC: of the finalists' second scores;
// CHAIN: they are one sum in the order of the coordinates, as the vector unit's scan and all inner products have it, and not four short
// ones, as behind the matrix cores' squared distances: reading halves makes no difference to what is returned.
template <int ST, bool HALVES, int METRIC, bool CHAIN>
__device__ __forceinline__ void select_query(const Dev &D, int nq, int k, const float *__restrict__ Q, const SearchScratch &S,
                                             float *__restrict__ out_dist, int64_t *__restrict__ out_ids) {
  __shared__ SelectShared sh;
  __shared__ uint32_t skey[kSurvivorCap];
  __shared__ uint32_t sidx[kSurvivorCap];
  __shared__ uint32_t scount;
  // Behind halves several workgroups may share a query's finalists (part of parts): a finalist's second score reads 16 bytes of a
  // line of memory for every four coordinates, 0.4 G such a second for a compute unit, and most of them idle where the
  // queries are few (64 queries, 170 to 250 finalists of 768 dimensions each: 113 us with one workgroup to a query).  Every one of
  // them takes the records and has a limit of its own; a finalist is scored by the one its place in the pool falls to, and the last one
  // to finish sorts what all have scored.
  const int part = HALVES ? (int)blockIdx.x / nq : 0, parts = HALVES ? (int)gridDim.x / nq : 1;
  const int q = HALVES ? (int)blockIdx.x - part * nq : (int)blockIdx.x;
  const int n = (int)*rec_count(S, (uint32_t)q);
  const unsigned long long base = S.qbase[q];
  const uint32_t *rk = rec_keys_of(S, base), *rp = rec_poss_of(S, base);
  const int metric = D.metric;
  const int lane = threadIdx.x & (kWave - 1);
  if (threadIdx.x == 0) scount = 0;
  __syncthreads();
  // (what they have scored goes behind the records, where there is room for it)
  const bool from_halves = HALVES && halves_exact_for(D, S, (uint32_t)q);
  const bool shared = HALVES && parts > 1 && !from_halves && (int64_t)n * D.d4 >= kSharedWork &&
                      S.qtotal[q] >= (uint32_t)n + 2u * kMaxK;
  if (HALVES && part > 0 && !shared) {  // uniform
    if (threadIdx.x == 0) overflow_request_done(S, gridDim.x);
    return;
  }
  auto mine = [&](uint32_t slot) { return !HALVES || !shared || (slot * 2654435761u >> 16) % (uint32_t)parts == (uint32_t)part; };

  // The records are taken into LDS in portions.  Once LDS is more than half full the k-th best
  // of what it holds becomes the limit (it cannot be better than the final k-th best): what is
  // worse is dropped, and later portions are filtered on the way in.  Under a limit only a few
  // per cent of a portion pass as a rule, so a portion is four times what LDS could take if all
  // of it passed; should it not fit after all, what it added is dropped, the limit is renewed
  // and the portion is read again, cut to what fits for certain.  Ties that no limit can
  // separate (LDS stays more than half full) are left to the selection in place below.
  // With norm-form scores among the records (flat lists under L2 scored on the matrix cores) a
  // limit taken from the k-th best record is loosened twice: once to bound the k-th best direct-form
  // score from above, once more to admit every record whose direct-form score may reach that.
  // Squared distances from halves: the same with their margin.  Inner products from halves are lower bounds of the negated
  // inner products, each with a margin of its own: a limit is the worst inner product of the k best such, from the floats
  // (limit_of_scored).
  const bool approx = HALVES || uses_norm_form(D);
  constexpr bool kScoredLimit = HALVES && METRIC == 1;
  const float slack = norm_form_slack(D.d), qn = !HALVES && approx ? S.qnorm[q] : 0.f;
  auto hq = [&]() { return half_query(D, S, (uint32_t)q); };  // (read where it is wanted: registers are short here)
  auto limit_from = [&](uint32_t kth) {
    if (HALVES) return halves_reach_key(D, halves_reach_key(D, kth, hq()), hq());
    return approx ? loosened_key(loosened_key(kth, slack, qn), slack, qn) : kth;
  };
  // a record's place in the pool (slot_of) -> which block, which place in it
  auto locate = [&](int i, uint32_t &b, uint32_t &moff) {
    b = (uint32_t)i / (uint32_t)D.T_m;
    moff = (uint32_t)i - b * (uint32_t)D.T_m;
  };
  auto id_of = [&](int i) -> int64_t {
    uint32_t b, moff;
    locate(i, b, moff);
    return block_ids(D, b)[moff];
  };
  // Where the halves beside the lists are the floats, the finalists are scored from those: a vector's chunks lie side by side by fours
  // there, where 16 bytes of the lists are a line of memory each.
  const float ixs = HALVES ? 1.f / halves_scale(D) : 1.f;
  auto half_floats = [&](const uint2 &h) {
    const float4 f = chunk_piece<1>(make_float4(__uint_as_float(h.x), __uint_as_float(h.y), 0.f, 0.f), 0);
    return make_float4(f.x * ixs, f.y * ixs, f.z * ixs, f.w * ixs);
  };
  auto half_chunk = [&](uint32_t b, uint32_t moff, int c) -> uint2 {  // chunk c of four floats
    return *reinterpret_cast<const uint2 *>(block_halves(D, b) + half_chunk_at(D, moff, (uint32_t)c >> 1) + (c & 1) * 8);
  };
  auto key_from_halves = [&](uint32_t b, uint32_t moff) __attribute__((always_inline)) -> uint32_t {  // squared distances, as direct_key has them
    const int sub = (int)(threadIdx.x & 3u);
    const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
    float acc = 0.f;
    for (int c0 = sub; c0 < D.d4; c0 += 32) {
      uint2 h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) h[u] = half_chunk(b, moff, min(c0 + 4 * u, D.d4 - 1));
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + 4 * u < D.d4) accumulate<0>(acc, half_floats(h[u]), y[c0 + 4 * u]);
    }
    acc += quad_xor<1>(acc);
    acc += quad_xor<2>(acc);
    return key_of_float(acc + 0.0f);
  };
  // The same for lists of halves and bytes: lane s of the four takes the 16-byte chunks s, s + 4, ...
  auto narrow_key = [&](uint32_t b, uint32_t moff) __attribute__((always_inline)) -> uint32_t {
    const int sub = (int)(threadIdx.x & 3u), vc = D.vchunks;
    const float4 *__restrict__ x = block_vecs(D, b) + (size_t)(moff / kWave) * vc * kWave + (moff & (kWave - 1));
    const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
    float acc = 0.f;
    for (int c0 = sub; c0 < vc; c0 += 16) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = x[(size_t)(c0 + 4 * u < vc ? c0 + 4 * u : c0) * kWave];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = c0 + 4 * u;
        if (c >= vc) break;
#pragma unroll
        for (int p = 0; p < pieces_of(ST); ++p) accumulate<METRIC>(acc, chunk_piece<ST>(v[u], p), y[pieces_of(ST) * c + p]);
      }
    }
    acc += quad_xor<1>(acc);
    acc += quad_xor<2>(acc);
    return key_of_float((METRIC == 0 ? acc : -acc) + 0.0f);
  };
  // place in the pool -> key of the candidate's direct-form squared distance (inner products from halves: of its inner product).  Four neighbouring lanes share
  // a candidate (a vector's chunks of 4 dimensions lie 1 KiB apart: every chunk is a memory
  // transaction of its own, and this way all of them are in flight at once): lane s of the four
  // takes chunks s, s + 4, ..., and the four partial sums are added pairwise.  All four lanes call
  // this with the same place and get the key.
  // One sum in the order of the coordinates (CHAIN): every chunk's four products are added by the lane that has the chunk, and the
  // four take the sum over from it.
  auto direct_key = [&](int i, int64_t *id) -> uint32_t {
    uint32_t b, moff;
    locate(i, b, moff);
    const int sub = (int)(threadIdx.x & 3u);
    if (id && sub == 0) *id = block_ids(D, b)[moff];
    if (CHAIN) {
      const float4 *__restrict__ x = block_vecs(D, b) + (size_t)(moff / kWave) * D.d4 * kWave + (moff & (kWave - 1));
      const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
      float acc = 0.f;
      for (int c0 = 0; c0 < D.d4; c0 += 32) {  // uniform
        float4 v[8], w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int c = min(c0 + 4 * u + sub, D.d4 - 1);
          v[u] = from_halves ? half_floats(half_chunk(b, moff, c)) : x[(size_t)c * kWave];
          w[u] = y[c];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          auto add = [&](auto lane_of) {
            constexpr int kLane = decltype(lane_of)::value;
            if (c0 + 4 * u + kLane >= D.d4) return;  // uniform
            float t = acc;
            accumulate<METRIC>(t, v[u], w[u]);
            acc = quad_broadcast<kLane>(t);
          };
          add(std::integral_constant<int, 0>{});
          add(std::integral_constant<int, 1>{});
          add(std::integral_constant<int, 2>{});
          add(std::integral_constant<int, 3>{});
        }
      }
      return key_of_float((METRIC == 0 ? acc : -acc) + 0.0f);
    }
    if (ST != 0) return narrow_key(b, moff);
    if (HALVES && from_halves) return key_from_halves(b, moff);  // uniform
    const float4 *__restrict__ x =
        block_vecs(D, b) + (size_t)(moff / kWave) * D.d4 * kWave + (moff & (kWave - 1));
    const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
    float acc = 0.f;
    int c = sub;
    for (; c + 28 < D.d4; c += 32) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = x[(size_t)(c + 4 * u) * kWave];
#pragma unroll
      for (int u = 0; u < 8; ++u) accumulate<METRIC>(acc, v[u], y[c + 4 * u]);
    }
    for (; c < D.d4; c += 4) accumulate<METRIC>(acc, x[(size_t)c * kWave], y[c]);
    acc += quad_xor<1>(acc);
    acc += quad_xor<2>(acc);
    return key_of_float((METRIC == 0 ? acc : -acc) + 0.0f);
  };
  // ... with sixteen neighbouring lanes to a candidate, where there are few: a lane has a quarter as many chunks, so a wide vector is a
  // turn or two of trips to memory and not a row of them (64 queries of 768 dimensions: the selection 92 us with four lanes, 80 with these, 73 by half as many
  // workgroups to a query; what is left of it is
  // mostly the 170 to 250 finalists of a query, 192 pieces of 16 bytes each from lines of their own).
  auto direct_key_row = [&](int i, int64_t *id) __attribute__((always_inline)) -> uint32_t {
    uint32_t b, moff;
    locate(i, b, moff);
    const int sub = (int)(threadIdx.x & 15u);
    if (sub == 0) *id = block_ids(D, b)[moff];
    const float4 *__restrict__ x = block_vecs(D, b) + (size_t)(moff / kWave) * D.d4 * kWave + (moff & (kWave - 1));
    const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
    float acc = 0.f;
    for (int c0 = 0; c0 < D.d4; c0 += 128) {  // uniform
      float4 v[8], w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = min(c0 + 16 * u + sub, D.d4 - 1);
        v[u] = from_halves ? half_floats(half_chunk(b, moff, c)) : x[(size_t)c * kWave];
        w[u] = y[c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (c0 + 16 * u >= D.d4) break;  // uniform
        auto add = [&](auto lane_of) {
          constexpr int kLane = decltype(lane_of)::value;
          if (c0 + 16 * u + kLane >= D.d4) return;  // uniform
          float t = acc;
          accumulate<METRIC>(t, v[u], w[u]);
          acc = row_broadcast<kLane>(t);
        };
        add(std::integral_constant<int, 0>{}); add(std::integral_constant<int, 1>{}); add(std::integral_constant<int, 2>{});
        add(std::integral_constant<int, 3>{}); add(std::integral_constant<int, 4>{}); add(std::integral_constant<int, 5>{});
        add(std::integral_constant<int, 6>{}); add(std::integral_constant<int, 7>{}); add(std::integral_constant<int, 8>{});
        add(std::integral_constant<int, 9>{}); add(std::integral_constant<int, 10>{}); add(std::integral_constant<int, 11>{});
        add(std::integral_constant<int, 12>{}); add(std::integral_constant<int, 13>{}); add(std::integral_constant<int, 14>{});
        add(std::integral_constant<int, 15>{});
      }
    }
    return key_of_float((METRIC == 0 ? acc : -acc) + 0.0f);
  };
  // The same for two candidates at once: both block look-ups go out together, then all the chunks of
  // both (a candidate is a chain of two round trips to memory; two of them side by side cost one).
  auto direct_key_pair = [&](int ia, int ib, int64_t *ida, int64_t *idb, uint32_t &ka, uint32_t &kb) {
    uint32_t ba, ma, bb, mb;
    locate(ia, ba, ma);
    locate(ib, bb, mb);
    const int sub = (int)(threadIdx.x & 3u);
    if (sub == 0) {
      *ida = block_ids(D, ba)[ma];
      *idb = block_ids(D, bb)[mb];
    }
    if (HALVES && from_halves) {  // uniform
      ka = key_from_halves(ba, ma);
      kb = key_from_halves(bb, mb);
      return;
    }
    if (ST != 0) {
      ka = narrow_key(ba, ma);
      kb = narrow_key(bb, mb);
      return;
    }
    const float4 *__restrict__ xa = block_vecs(D, ba) + (size_t)(ma / kWave) * D.d4 * kWave + (ma & (kWave - 1));
    const float4 *__restrict__ xb = block_vecs(D, bb) + (size_t)(mb / kWave) * D.d4 * kWave + (mb & (kWave - 1));
    const float4 *__restrict__ y = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d);
    float acca = 0.f, accb = 0.f;
    int c = sub;
    for (; c + 28 < D.d4; c += 32) {
      float4 va[8], vb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) va[u] = xa[(size_t)(c + 4 * u) * kWave];
#pragma unroll
      for (int u = 0; u < 8; ++u) vb[u] = xb[(size_t)(c + 4 * u) * kWave];
#pragma unroll
      for (int u = 0; u < 8; ++u) accumulate<METRIC>(acca, va[u], y[c + 4 * u]);
#pragma unroll
      for (int u = 0; u < 8; ++u) accumulate<METRIC>(accb, vb[u], y[c + 4 * u]);
    }
    for (; c < D.d4; c += 4) {
      const float4 va = xa[(size_t)c * kWave], vb = xb[(size_t)c * kWave];
      accumulate<METRIC>(acca, va, y[c]);
      accumulate<METRIC>(accb, vb, y[c]);
    }
    acca += quad_xor<1>(acca);
    acca += quad_xor<2>(acca);
    accb += quad_xor<1>(accb);
    accb += quad_xor<2>(accb);
    ka = key_of_float((METRIC == 0 ? acca : -acca) + 0.0f);
    kb = key_of_float((METRIC == 0 ? accb : -accb) + 0.0f);
  };
  // A limit from any k or more candidates (sh.pay[0 .. m), at most kMaxK): no final k-th best is worse than the worst of them.
  __shared__ uint32_t s_worst;
  auto limit_of_scored = [&](int m) -> uint32_t {
    if (threadIdx.x == 0) s_worst = 0u;
    __syncthreads();
    uint32_t worst = 0u;
    for (int p0 = 0; p0 < m; p0 += kTopkThreads / 4) {  // uniform trip count
      const int p = p0 + (int)(threadIdx.x >> 2);
      const uint32_t key = direct_key((int)sh.pay[p < m ? p : m - 1], nullptr);
      worst = key > worst ? key : worst;
    }
    worst = wave_reduce_last(worst, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
    if (lane == kWave - 1) atomicMax(&s_worst, worst);
    __syncthreads();
    return halves_reach_ip_key(s_worst, hq());
  };
  // ... namely those of `count` records whose keys are not worse than T, which k or more are
  auto limit_below = [&](int count, uint32_t T, auto key, auto item) -> uint32_t {
    if (threadIdx.x == 0) sh.cnt[0] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < count; j += kTopkThreads)
      if (key(j) <= T) {
        const uint32_t p = atomicAdd(&sh.cnt[0], 1u);
        if (p < (uint32_t)kMaxK) sh.pay[p] = (uint32_t)item(j);
      }
    __syncthreads();
    return limit_of_scored(min((int)sh.cnt[0], kMaxK));
  };
  // what LDS holds is cut down to the records not worse than the limit: everybody reads its
  // entries, then everybody writes the kept ones back
  auto keep_not_worse = [&](int have, uint32_t lim) {
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));  // (addresses made from it are not kept from one use of this to the next)
    constexpr int kMine = kSurvivorCap / kTopkThreads;
    uint32_t mk[kMine], mi[kMine];
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int j = tid + u * kTopkThreads;
      mk[u] = j < have ? skey[j] : 0xFFFFFFFFu;
      mi[u] = j < have ? sidx[j] : 0u;
    }
    __syncthreads();
    if (threadIdx.x == 0) scount = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int j = tid + u * kTopkThreads;
      const bool keep = j < have && mk[u] <= lim;
      const unsigned long long mask = __ballot(keep);
      if (mask) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&scount, (uint32_t)__popcll(mask));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        if (keep) {
          const uint32_t slot = at + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
          skey[slot] = mk[u];
          sidx[slot] = mi[u];
        }
      }
    }
    __syncthreads();
  };
  uint32_t limit = S.bound[q];
  if (HALVES) limit = halves_bound_key(D, limit, hq());
  bool in_lds = true;
  // (halves that are not finite among the records: none of the keys is gone by)
  const bool flagged = HALVES && *rec_flag(S, (uint32_t)q) != 0u;
  if (flagged) { limit = 0xFFFFFFFFu; in_lds = false; }
  __shared__ uint32_t s_over;
  int stretch = 1;  // portions as a multiple of the room in LDS
  // More records than LDS holds (the query's bound was loose: its sample did not look like its
  // candidates): a first limit comes from a pilot, every (n / pilot)-th record, so that the
  // records are filtered from the first portion on instead of filling LDS once unfiltered.  A query
  // with tens of thousands of records (a hot list) takes a pilot as large as LDS: the k-th best of
  // 4096 lets about k / 4096 of the records pass, which fit in one go.
  constexpr int kPilot = 1024;
  if (!flagged && n > kSurvivorCap && k <= kPilot) {  // uniform over the workgroup
    const int pilot = n >= 8 * kSurvivorCap ? kSurvivorCap : kPilot;
    const int stride = n / pilot;
    for (int j = threadIdx.x; j < pilot; j += kTopkThreads) skey[j] = rk[(size_t)j * stride];
    __syncthreads();
    const SelectResult r = wg_radix_select<32>(
        pilot, (uint32_t)k, [&](int j, uint64_t &kv) { kv = skey[j]; return true; }, sh.hist, sh.bc, (uint32_t)(k + k / 16));
    uint32_t lim;
    if constexpr (kScoredLimit)
      lim = limit_below(pilot, (uint32_t)r.T, [&](int j) { return skey[j]; }, [&](int j) { return (int)rp[(size_t)j * stride]; });
    else lim = limit_from((uint32_t)r.T);
    limit = lim < limit ? lim : limit;
    stretch = pilot == kSurvivorCap ? 16 : 4;
    __syncthreads();  // the pilot's keys are done with
  }
  // A query whose records take several round trips to stream keeps, of a record that passes, its
  // index first and fetches the positions of what LDS holds in the end (the positions of the many
  // that do not pass are never read); a query that is through in one round trip loads both together.
  // 16 keys in flight per thread either way (24 or 32 take the kernel past 128 registers).
  const bool deferred = n > 16 * kTopkThreads;  // uniform over the workgroup
  auto stream = [&](auto tag, int next, int m) {
    constexpr bool kDeferred = decltype(tag)::value;
    constexpr int kInFlight = kDeferred ? 16 : 16;
    for (int j0 = 0; j0 < m; j0 += kInFlight * kTopkThreads) {
      uint32_t kv[kInFlight], pv[kDeferred ? 1 : kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {  // clamped index: the loads are unconditional and issue back to back
        const int j = j0 + u * kTopkThreads + (int)threadIdx.x;
        kv[u] = rk[next + (j < m ? j : m - 1)];
      }
      if (!kDeferred) {
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
          const int j = j0 + u * kTopkThreads + (int)threadIdx.x;
          pv[u] = rp[next + (j < m ? j : m - 1)];
        }
      }
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int j = j0 + u * kTopkThreads + (int)threadIdx.x;
        const bool keep = j < m && kv[u] <= limit;
        const unsigned long long mask = __ballot(keep);
        if (mask) {  // uniform over the wavefront
          uint32_t at = 0;
          if (lane == 0) at = atomicAdd(&scount, (uint32_t)__popcll(mask));
          at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
          if (keep) {
            const uint32_t slot = at + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
            if (slot < (uint32_t)kSurvivorCap) { skey[slot] = kv[u]; sidx[slot] = kDeferred ? (uint32_t)(next + j) : pv[kDeferred ? 0 : u]; }
            else s_over = 1u;
          }
        }
      }
    }
  };
  // Records that all fit are taken as they come: every one of them passed the query's bound in the scan.  (Through the
  // filter below, a count and a reservation per 64 of them, they cost the selection two microseconds more.)
  int next = flagged ? n : 0;
  if (!flagged && n <= kSurvivorCap) {
    constexpr int kMine = kSurvivorCap / kTopkThreads;
    uint32_t kv[kMine], pv[kMine];
    const int last = n > 0 ? n - 1 : 0;
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int j = (int)threadIdx.x + u * kTopkThreads;
      if (u * kTopkThreads < n) { kv[u] = rk[j < n ? j : last]; pv[u] = rp[j < n ? j : last]; }  // uniform
    }
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int j = (int)threadIdx.x + u * kTopkThreads;
      if (j < n) { skey[j] = kv[u]; sidx[j] = pv[u]; }
    }
    if (threadIdx.x == 0) scount = (uint32_t)n;
    next = n;
    __syncthreads();
  }
  while (next < n) {  // every branch here is uniform over the workgroup
    const int count = (int)scount;
    const int m = min(n - next, stretch * (kSurvivorCap - count));
    if (threadIdx.x == 0) s_over = 0;
    __syncthreads();
    // (the positions come with the keys, or afterwards, but never from inside the filter loop: a load
    // there, for the records that pass, would make every turn of it a round trip of its own)
    if (deferred) stream(std::true_type{}, next, m);
    else stream(std::false_type{}, next, m);
    __syncthreads();
    const bool over = s_over != 0;
    __syncthreads();
    if (over) {  // did not fit: forget what this portion added; below, the limit is renewed from the rest
      if (threadIdx.x == 0) scount = (uint32_t)count;
      __syncthreads();
    } else {
      next += m;
      if (next >= n) break;
    }
    const int have = (int)scount;
    if (!over && have <= kSurvivorCap / 2) continue;
    if (have >= k) {
      // tighten
      const SelectResult r = wg_radix_select<32>(
          have, (uint32_t)k, [&](int j, uint64_t &kv) { kv = skey[j]; return true; }, sh.hist, sh.bc, (uint32_t)(k + k / 16));
      uint32_t lim;
      if constexpr (kScoredLimit)
        lim = limit_below(have, (uint32_t)r.T, [&](int j) { return skey[j]; },
                          [&](int j) { return deferred ? (int)rp[sidx[j]] : (int)sidx[j]; });
      else lim = limit_from((uint32_t)r.T);
      limit = lim < limit ? lim : limit;
      keep_not_worse(have, limit);  // drop what is worse
      if ((int)scount > kSurvivorCap / 2) { in_lds = false; break; }
    }
    // from the first limit on, portions may be stretched; a portion that did not fit is read
    // again unstretched (it fits then, whatever it holds)
    stretch = over ? 1 : 4;
  }

  if (deferred && in_lds) {  // uniform: LDS holds indices of records; now their places in the pool
    __syncthreads();
    const int have = (int)scount;
    for (int j = threadIdx.x; j < have; j += kTopkThreads) sidx[j] = rp[sidx[j]];
    __syncthreads();
  }
  int kk = -1;
  if (approx && in_lds) {  // uniform over the workgroup
    // The usual case: the finalists (every record that may be among the k best by direct-form
    // scores, i.e. not worse than the twice loosened k-th best of what LDS holds) number little
    // more than k.  They get their direct-form scores and ids in one go and are sorted by those.
    const int have = (int)scount;
    uint32_t lim = 0xFFFFFFFFu;
    if (have > k) {
      const SelectResult r = wg_radix_select<32>(
          have, (uint32_t)k, [&](int j, uint64_t &kv) { kv = skey[j]; return true; }, sh.hist, sh.bc, (uint32_t)(k + k / 16));
      lim = kScoredLimit ? (uint32_t)r.T : limit_from((uint32_t)r.T);
      if (!kScoredLimit) limit = lim < limit ? lim : limit;
    }
    if (threadIdx.x == 0) sh.cnt[0] = 0;
    __syncthreads();
    auto collect = [&](bool all, uint32_t above, uint32_t upto, bool share) {  // records whose keys are in (above, upto]
      for (int j = threadIdx.x; j < have; j += kTopkThreads)
        if (skey[j] <= upto && (all || skey[j] > above) && (!share || mine(sidx[j]))) {
          const uint32_t p = atomicAdd(&sh.cnt[0], 1u);
          if (p < (uint32_t)kMaxK) sh.pay[p] = sidx[j];
        }
      __syncthreads();
    };
    uint32_t worst = 0u;
    auto score = [&](int from, int m) {  // finalists from .. m - 1
      constexpr int kFours = kTopkThreads / 4;
      for (int p0 = from; p0 < m;) {  // uniform trip count: the lanes of a four stay together
        const int p = p0 + (int)(threadIdx.x >> 2);
        if (CHAIN && m - p0 <= kTopkThreads / 16) {  // uniform
          const int pr = p0 + (int)(threadIdx.x >> 4);
          int64_t id = 0;
          const uint32_t key = direct_key_row((int)sh.pay[pr < m ? pr : m - 1], &id);
          if (kScoredLimit) worst = max(worst, key);
          if (pr < m && (threadIdx.x & 15u) == 0) {
            sh.k1[pr] = key;
            sh.k2[pr] = (uint64_t)id ^ 0x8000000000000000ull;
          }
          break;
        }
        if (!CHAIN && m - p0 > kFours) {  // uniform: every four takes two finalists, p and p + kFours
          const int p2 = p + kFours;
          int64_t id = 0, id2 = 0;
          uint32_t key, key2;
          direct_key_pair((int)sh.pay[p < m ? p : m - 1], (int)sh.pay[p2 < m ? p2 : m - 1], &id, &id2, key, key2);
          if ((threadIdx.x & 3u) == 0) {
            if (p < m) { sh.k1[p] = key; sh.k2[p] = (uint64_t)id ^ 0x8000000000000000ull; }
            if (p2 < m) { sh.k1[p2] = key2; sh.k2[p2] = (uint64_t)id2 ^ 0x8000000000000000ull; }
          }
          p0 += 2 * kFours;
        } else {
          int64_t id = 0;
          const uint32_t key = direct_key((int)sh.pay[p < m ? p : m - 1], &id);
          if (kScoredLimit) worst = max(worst, key);
          if (p < m && (threadIdx.x & 3u) == 0) {
            sh.k1[p] = key;
            sh.k2[p] = (uint64_t)id ^ 0x8000000000000000ull;
          }
          p0 += kFours;
        }
      }
    };
    collect(true, 0u, lim, !kScoredLimit || have <= k);
    int m = (int)sh.cnt[0];  // (a shared query's k best are scored by all of its workgroups)
    if (m <= kMaxK) {
      score(0, m);
      if constexpr (kScoredLimit) {
        // the k best by what halves say are scored: whatever may still be better than the worst of them is scored as well
        if (have > k) {  // uniform
          worst = wave_reduce_last(worst, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
          if (threadIdx.x == 0) s_worst = 0u;
          __syncthreads();
          if (lane == kWave - 1) atomicMax(&s_worst, worst);
          __syncthreads();
          const uint32_t upto = halves_reach_ip_key(s_worst, hq());
          limit = upto < limit ? upto : limit;
          if (upto > lim) collect(false, lim, upto, true);
          const int more = (int)sh.cnt[0];
          if (more <= kMaxK) score(m, more);
          m = more;
        }
      }
      if (!shared && m <= kMaxK) {
        wg_sort<32>(m, sh.k1, sh.k2, sh.pay);
        kk = k < m ? k : m;
      }
    }
    if (HALVES && shared) {  // uniform
      __syncthreads();
      if (m > kMaxK) {
        if (threadIdx.x == 0) __hip_atomic_store(rec_alone(S, (uint32_t)q), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        // What is handed over are the workgroup's own of all it has scored.  (Whose a finalist is cannot go by a threshold: where
        // more than kMaxK records offered themselves for a limit, the workgroups have limits, and so thresholds, of their own.)
        constexpr int kMine = kMaxK / kTopkThreads;
        uint32_t slot[kMine];
        if (threadIdx.x == 0) sh.cnt[1] = 0u;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kMine; ++u) {
          const int p = (int)threadIdx.x + u * kTopkThreads;
          slot[u] = p < m && mine(sh.pay[p]) ? atomicAdd(&sh.cnt[1], 1u) : ~0u;
        }
        __syncthreads();
        if (threadIdx.x == 0) sh.bc[0] = sh.cnt[1] ? atomicAdd(rec_scored(S, (uint32_t)q), sh.cnt[1]) : 0u;
        __syncthreads();
        uint32_t *ok = const_cast<uint32_t *>(rk) + n, *op = const_cast<uint32_t *>(rp) + n;
#pragma unroll
        for (int u = 0; u < kMine; ++u) {
          const int p = (int)threadIdx.x + u * kTopkThreads;
          const uint32_t o = slot[u] == ~0u ? ~0u : sh.bc[0] + slot[u];
          if (o >= (uint32_t)kMaxK) continue;  // (too many all in all: the last workgroup sees that)
          __hip_atomic_store(&op[o], (uint32_t)sh.k1[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&ok[2 * o], (uint32_t)sh.k2[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&ok[2 * o + 1], (uint32_t)(sh.k2[p] >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
  if (HALVES && shared) {  // uniform
    if (!in_lds && threadIdx.x == 0) __hip_atomic_store(rec_alone(S, (uint32_t)q), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // what this wavefront has scored is out ...
    __syncthreads();                                  // ... and so is everybody's before the workgroup counts itself off
    if (threadIdx.x == 0) {
      sh.bc[0] = atomicAdd(rec_done(S, (uint32_t)q), 1u) + 1u == (uint32_t)parts;
      sh.bc[1] = __hip_atomic_load(rec_alone(S, (uint32_t)q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sh.bc[2] = __hip_atomic_load(rec_scored(S, (uint32_t)q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!sh.bc[0]) {  // uniform: the last one goes on
      if (threadIdx.x == 0) overflow_request_done(S, gridDim.x);
      return;
    }
    const int all = (int)sh.bc[2];
    if (!sh.bc[1] && all <= kMaxK) {  // (otherwise the last one goes on alone, from its own records)
      const uint32_t *ok = rk + n, *op = rp + n;
      for (int p = threadIdx.x; p < all; p += kTopkThreads) {
        sh.k1[p] = __hip_atomic_load(&op[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.k2[p] = (uint64_t)__hip_atomic_load(&ok[2 * p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) |
                   (uint64_t)__hip_atomic_load(&ok[2 * p + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) << 32;
        sh.pay[p] = 0u;
      }
      wg_sort<32>(all, sh.k1, sh.k2, sh.pay);
      kk = k < all ? k : all;
    }
  }
  if (approx && kk < 0) {  // uniform over the workgroup
    // Many finalists (near-ties by the thousand): whatever is not worse than the limit is scored
    // again where it lies, and the selection then runs on direct-form scores as for the other kinds of list.
    if (in_lds) {
      keep_not_worse((int)scount, limit);
      const int have = (int)scount;
      for (int j0 = 0; j0 < have; j0 += kTopkThreads / 4) {
        const int j = j0 + (int)(threadIdx.x >> 2);
        const uint32_t key = direct_key((int)sidx[j < have ? j : have - 1], nullptr);
        if (j < have && (threadIdx.x & 3u) == 0) skey[j] = key;
      }
    } else {
      if (HALVES && n > kSurvivorCap / 2 && threadIdx.x == 0) D.mirror->halves_failed = 1u;  // (halves_may_tell, rtams.hip)
      // the records are this query's own
      uint32_t *wk = const_cast<uint32_t *>(rk);
      for (int j0 = 0; j0 < n; j0 += kTopkThreads / 4) {
        const int j = j0 + (int)(threadIdx.x >> 2);
        const int jj = j < n ? j : n - 1;
        const bool want = rk[jj] <= limit;
        uint32_t key = 0xFFFFFFFFu;
        if (__any(want)) {  // uniform over the wavefront, so the fours stay together
          const uint32_t dk = direct_key((int)rp[jj], nullptr);
          key = want ? dk : key;
        }
        if (j < n && (threadIdx.x & 3u) == 0) wk[j] = key;
      }
    }
    __syncthreads();
  }
  if (kk < 0) {
    if (in_lds)
      kk = select_topk((int)scount, k, [&](int j) { return skey[j]; }, [&](int j) { return (int)sidx[j]; },
                       id_of, sh);
    else
      kk = select_topk(n, k, [&](int j) { return rk[j]; }, [&](int j) { return (int)rp[j]; }, id_of, sh);
  }

  for (int r = threadIdx.x; r < k; r += kTopkThreads) {
    size_t o = (size_t)q * k + r;
    if (r < kk) {
      out_dist[o] = score_of_key((uint32_t)sh.k1[r], metric);
      out_ids[o] = (int64_t)(sh.k2[r] ^ 0x8000000000000000ull);
    } else {
      out_dist[o] = metric == 0 ? __builtin_inff() : -__builtin_inff();
      out_ids[o] = -1;
    }
  }
  if (q == 0 && threadIdx.x == 0) *S.cursor = 0ull;  // the next request on this slice finds its records' room free
  // the records are not looked at any more (the selection ended with a barrier)
  if (threadIdx.x == 0) overflow_request_done(S, gridDim.x);
}

template <int ST>
__global__ __launch_bounds__(kTopkThreads, 4) void k_select(Dev D, int k, const float *__restrict__ Q, SearchScratch S,
                                                        float *__restrict__ out_dist, int64_t *__restrict__ out_ids) {
  select_query<ST, false, 0, false>(D, 0, k, Q, S, out_dist, out_ids);
}
template <int METRIC, bool CHAIN>
__global__ __launch_bounds__(kTopkThreads, 4) void k_select_halves(Dev D, int nq, int k, const float *__restrict__ Q, SearchScratch S,
                                                        float *__restrict__ out_dist, int64_t *__restrict__ out_ids) {
  select_query<0, true, METRIC, CHAIN>(D, nq, k, Q, S, out_dist, out_ids);
}

void launch_select(const Dev &D, int64_t nq, int k, const float *Q, const SearchScratch &S, float *out_dist, int64_t *out_ids,
                   hipStream_t s) {
  if (nq <= 0) return;
  if (D.scan_halves) {
    // as many to a query as give no compute unit two workgroups: each reads all of the query's records, so twice as many
    // cost more than they bring (256 queries over 20 M x 256, skewed 174 / 206 us, 64 over 5 M x 768 73 / 77).  Whole requests
    // whose finalists are shared, k 100 to 128 of 64 probes, over 1 M x 256, 500 k x 768 and 200 k x 1,536, both metrics: at 32 to
    // 128 queries half as many 1.02 times as long on average (up to 1.09), twice as many 1.06 (1.19), four times 1.26; one more
    // than fits, for a number that does not divide (40 to 240 queries), 1.06 (1.14).  Of 32 queries and fewer eight workgroups are as good as 16.
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(kComputeUnits / nq, kSelectParts));
    const auto kernel = D.metric != 0 ? k_select_halves<1, true> : D.scan_mfma ? k_select_halves<0, false> : k_select_halves<0, true>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nq * parts)), dim3(kTopkThreads), 0, s, D, (int)nq, k, Q, S, out_dist, out_ids);
    return;
  }
  typedef void (*Kernel)(Dev, int, const float *, SearchScratch, float *, int64_t *);
  static const Kernel kernels[3] = {k_select<0>, k_select<1>, k_select<2>};
  hipLaunchKernelGGL(kernels[D.storage], dim3((unsigned)nq), dim3(kTopkThreads), 0, s, D, k, Q, S, out_dist, out_ids);
}

}  // namespace rtams
