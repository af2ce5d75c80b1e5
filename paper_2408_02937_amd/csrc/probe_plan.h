// Probe selection and the per-query plan of a search request, by one workgroup per query.
#pragma once
#include "search_common.h"

namespace rtams {

// ------------------------------------------------------------ probe and plan
// One workgroup per query: the nprobe best centroids by (score, index), best
// first; then the plan of the scan: the visible length of each probed list is
// read ONCE here, so that scan and selection agree on it whatever an insertion
// publishes meanwhile, and the query gets its slice of the candidate array.
// FROM_APPROX: the request's coarse scores are fp32 approximations from the
// matrix cores (coarse_mfma.hip).  The nprobe-th smallest of them plus the error
// band bounds every centroid that can be among the exact nprobe best; those
// candidates are scored in the fixed double arithmetic here and ordered
// exactly.  If the band holds more candidates than LDS, the whole row is scored
// exactly instead (what small requests, which skip the matrix cores, always do).
// MINE: scores of the row a thread holds in registers, 0 for rows too long for that.  A row that is held is read once,
// all its loads in flight together; every pass of a selection that reads the row again is a chain of trips to memory
// (16,384 lists: 25 us for the selection alone, most of it such passes).
// DIRECT: a small request whose scan goes straight from the probes (small.hip).  The scores were written by other
// workgroups of this very kernel, and the pairs are not counted by list but stand as they are, query after query.
template <bool FROM_APPROX>
struct ProbeShared {
  __attribute__((aligned(8))) uint32_t hist[kSelectLdsWords];
  uint32_t bc[4];
  uint32_t cnt[2];
  uint64_t k1[kMaxNprobe];
  uint64_t k2[kMaxNprobe];
  uint32_t pay[kMaxNprobe];
  float4 yv[FROM_APPROX ? 512 : 1];  // the query (d <= 2048)
};
template <bool FROM_APPROX, int MINE, bool DIRECT>
__device__ __forceinline__ void probe_plan(const Dev &D, int64_t nq, int q, int nprobe, int max_nprobe, const SearchScratch &S,
                                           const float *__restrict__ Q, int32_t *probe_out, ProbeShared<FROM_APPROX> &sh) {
  uint32_t *hist = sh.hist, *bc = sh.bc, *cnt = sh.cnt, *pay = sh.pay;
  uint64_t *k1 = sh.k1, *k2 = sh.k2;
  float4 *yv = sh.yv;
  const int T = (int)blockDim.x;
  const int n = D.nlist;
  double *sc = S.scores + (size_t)q * n;
  const int metric = D.metric;
  // the fixed arithmetic of coarse.hip for one centroid: a chain of multiply-adds in the order of the
  // coordinates, fed by 16-byte loads of which one set of eight is in flight while the other is used up (one
  // coordinate per load, each waited for, made a candidate of 768 dimensions cost a hundred nanoseconds per
  // coordinate; one set at a time, a trip to memory per eight chunks).  The query comes out of LDS.
  auto exact = [&](int c) __attribute__((always_inline)) -> double {
    const float4 *r4 = reinterpret_cast<const float4 *>(D.centroids + (size_t)c * D.d);
    const int d4 = D.d4;
    double acc = 0.0;
    auto chain = [&](const float4 &y, const float4 &r) {
      if (metric == 0) {
        const double t0 = (double)y.x - (double)r.x; acc = __builtin_fma(t0, t0, acc);
        const double t1 = (double)y.y - (double)r.y; acc = __builtin_fma(t1, t1, acc);
        const double t2 = (double)y.z - (double)r.z; acc = __builtin_fma(t2, t2, acc);
        const double t3 = (double)y.w - (double)r.w; acc = __builtin_fma(t3, t3, acc);
      } else {
        acc = __builtin_fma((double)y.x, (double)r.x, acc);
        acc = __builtin_fma((double)y.y, (double)r.y, acc);
        acc = __builtin_fma((double)y.z, (double)r.z, acc);
        acc = __builtin_fma((double)y.w, (double)r.w, acc);
      }
    };
    float4 sa[8], sb[8];
    auto load = [&](float4 *set, int j) {
#pragma unroll
      for (int u = 0; u < 8; ++u) set[u] = r4[j + u];
      __builtin_amdgcn_sched_barrier(0);  // the loads go out here
    };
    auto use = [&](const float4 *set, int j) {
#pragma unroll
      for (int u = 0; u < 8; ++u) chain(yv[j + u], set[u]);
      __builtin_amdgcn_sched_barrier(0);
    };
    int j = 0;
    if (d4 >= 8) load(sa, 0);
    for (; j + 24 <= d4; j += 16) {
      load(sb, j + 8);
      use(sa, j);
      load(sa, j + 16);
      use(sb, j + 8);
    }
    if (j + 16 <= d4) { load(sb, j + 8); use(sa, j); use(sb, j + 8); j += 16; }
    else if (j + 8 <= d4) { use(sa, j); j += 8; }
    for (; j < d4; ++j) chain(yv[j], r4[j]);
    return acc;
  };
  auto key_of_score = [&](double x) -> uint64_t {
    x = (metric == 0 ? x : -x) + 0.0;  // +0.0 folds -0 into +0
    return key_of_double(x);
  };
  if (FROM_APPROX) {
    for (int c = threadIdx.x; c < D.d4; c += T) yv[c] = reinterpret_cast<const float4 *>(Q + (size_t)q * D.d)[c];
    __syncthreads();
  }
  constexpr int kHeld = MINE > 0 ? MINE : 1;
  bool done = false;  // k1 / k2 / pay hold the nprobe winners, not yet sorted
  if (FROM_APPROX && nprobe < n) {
    const float *ap = S.approx + (size_t)q * n;
    float mine[kHeld];
    if (MINE > 0) {
#pragma unroll
      for (int u = 0; u < kHeld; ++u) mine[u] = ap[min((int)threadIdx.x + u * T, n - 1)];
    }
    auto each_approx = [&](auto body) {  // body(index, score)
      if (MINE > 0) {
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
          if ((int)threadIdx.x + u * T < n) body((int)threadIdx.x + u * T, mine[u]);
      } else {
        for (int i = threadIdx.x; i < n; i += T) body(i, ap[i]);
      }
    };
    const float band = search_row_meta(D, nq, S.qhalf)[q].band;  // 2 E, see coarse_mfma.hip
    // The candidates are sorted by their exact scores anyway, so the selection may stop at a threshold that admits some more
    // lists than nprobe; with the band they have to fit LDS, though, and where they turn out not to, but without those few
    // would, the threshold is taken exactly.  (256 queries over 16,384 lists of 64 dimensions, 980 probes: 243 us with the
    // early stop alone, whose candidates did not fit, so that the whole row was scored; 109 now.)
    uint32_t stop = min((uint32_t)(nprobe + nprobe / 8), (uint32_t)(nprobe + kMaxNprobe) / 2);
    int nc;
    for (;;) {  // uniform over the workgroup
      const SelectResult ra = wg_radix_select_each<32>(
          (uint32_t)nprobe, [&](auto body) { each_approx([&](int, float v) { body((uint64_t)key_of_float(v + 0.0f)); }); },
          hist, bc, stop);
      const uint32_t tk = (uint32_t)ra.T;  // key of (an upper bound of) the nprobe-th smallest approximation
      const float t = __uint_as_float((tk & 0x80000000u) ? (tk & 0x7fffffffu) : ~tk);
      const float limit = t + band;
      if (threadIdx.x == 0) cnt[0] = 0;
      __syncthreads();
      each_approx([&](int i, float v) {
        if (v <= limit) {
          uint32_t p = atomicAdd(&cnt[0], 1u);
          if (p < (uint32_t)kMaxNprobe) pay[p] = (uint32_t)i;
        }
      });
      __syncthreads();
      nc = (int)cnt[0];
      const int beyond = nc - (nprobe - (int)ra.need + (int)ra.c_eq);  // the band's own; a lower threshold has fewer of them
      if (nc <= kMaxNprobe || stop == 0u || nprobe + beyond - beyond / 4 > kMaxNprobe) break;
      stop = 0u;
    }
    if (nc >= nprobe && nc <= kMaxNprobe) {  // (fewer than nprobe: scores that do not compare, e.g. NaN)
      for (int p = threadIdx.x; p < nc; p += T) {
        const int c = (int)pay[p];
        k1[p] = key_of_score(exact(c));
        k2[p] = (uint64_t)c;
      }
      wg_sort<64>(nc, k1, k2, pay);  // by (exact score, index): the first nprobe are the answer
      done = true;
    }
  }
  SelectResult r1{~0ull, 0, 0}, r2{~0ull, 0, 0};
  const bool all = nprobe >= n;
  if (!done && FROM_APPROX) {  // the filter did not narrow it, or every list is probed: exact order of the whole row
    for (int i = threadIdx.x; i < n; i += T) sc[i] = exact(i);
    __syncthreads();
  }
  if (!done) {
  // (a request whose filter did not narrow the row down reads it from memory: that is rare, and the registers are taken)
  constexpr bool kHold = MINE > 0 && !FROM_APPROX;
  double held[kHeld];
  if (kHold) {
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      const double *at = &sc[min((int)threadIdx.x + u * T, n - 1)];
      held[u] = DIRECT ? __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *at;
    }
  }
  auto each_key = [&](auto body) {  // body(index, key)
    if (kHold) {
#pragma unroll
      for (int u = 0; u < kHeld; ++u)
        if ((int)threadIdx.x + u * T < n) body((int)threadIdx.x + u * T, key_of_score(held[u]));
    } else {
      for (int i = threadIdx.x; i < n; i += T) body(i, key_of_score(sc[i]));
    }
  };
  // The winners are sorted by (score, index): a threshold that admits a few more than nprobe does, the first nprobe are
  // taken behind the sort.  Only where ties leave more than that are they told apart by index first.
  // (Behind the filter this is rare, and the scalar registers are taken: exactly nprobe there.)
  const uint32_t room = (uint32_t)(FROM_APPROX ? nprobe : min(nprobe + 16, kMaxNprobe));
  if (!all) {
    r1 = wg_radix_select_each<64>((uint32_t)nprobe,
                                  [&](auto body) { each_key([&](int, uint64_t k) { body(k); }); }, hist, bc, FROM_APPROX ? 0u : room);
    if ((uint32_t)nprobe - r1.need + r1.c_eq > room)  // ties at the boundary go to the lower index
      r2 = wg_radix_select_each<32>(
          r1.need, [&](auto body) { each_key([&](int i, uint64_t k) { if (k == r1.T) body((uint64_t)(uint32_t)i); }); },
          hist, bc);
  }
  if (threadIdx.x == 0) cnt[0] = 0;
  __syncthreads();
  each_key([&](int i, uint64_t k) {
    bool take = all || k < r1.T || (k == r1.T && ((uint32_t)nprobe - r1.need + r1.c_eq <= room || (uint64_t)i <= r2.T));
    if (take) {
      uint32_t p = atomicAdd(&cnt[0], 1u);
      k1[p] = k; k2[p] = (uint64_t)i; pay[p] = (uint32_t)i;
    }
  });
  __syncthreads();
  wg_sort<64>(FROM_APPROX ? nprobe : (int)cnt[0], k1, k2, pay);
  }  // !done
  if (done) {  // the sort carried no payload: the list index is the second key
    __syncthreads();
    for (int p = threadIdx.x; p < nprobe; p += T) pay[p] = (uint32_t)k2[p];
    __syncthreads();
  }

  // plan
  int32_t *pl = S.probe_list + (size_t)q * max_nprobe;
  uint32_t *plen = S.probe_len + (size_t)q * max_nprobe;
  for (int p = threadIdx.x; p < nprobe; p += T) {
    int list = (int)pay[p];
    pl[p] = list;
    if (probe_out) probe_out[(size_t)q * nprobe + p] = list;
    uint32_t len = __hip_atomic_load(&D.visible_len[list], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    plen[p] = len;
    pay[p] = len;  // reuse as lengths for the prefix sum below
    // rank of this pair among the pairs that probe the same list (grouping for the scan)
    if (!DIRECT) S.pair_slot[(size_t)q * max_nprobe + p] = atomicAdd(&S.list_cnt[list], 1u);
  }
  __syncthreads();
  unsigned long long tot = 0;
  if (threadIdx.x < kWave) {
    for (int p = threadIdx.x; p < nprobe; p += kWave) tot += pay[p];
    tot = wave_running_sum(tot);  // of all, in the last lane
  }
  if (threadIdx.x == kWave - 1) {
    unsigned long long base = 0;
    if (probe_out) tot = 0;  // the probe hook: nothing is scanned afterwards, no room for records is taken
    if (tot > 0xFFFFFFFFull) tot = ~0ull;  // cannot be indexed: treated as overflow below
    if (tot != ~0ull) base = atomicAdd(S.cursor, tot);
    if (tot != ~0ull && base + tot > S.cand_cap) {  // does not fit into the slice any more: the shared reserve
      base = overflow_take(S, tot);
      if (base == ~0ull) tot = ~0ull;
    }
    if (tot == ~0ull) {  // not enough candidate scratch for this query
      base = 0;
      atomicCAS(&D.ctrl->search_error, 0, -6);
      D.mirror->search_error = -6;
      tot = 0;
      for (int p = 0; p < nprobe; ++p) plen[p] = 0;
    }
    S.qbase[q] = base;
    S.qtotal[q] = (uint32_t)tot;
    if (!DIRECT && D.nlist >= 32) S.done_count[q] = 0u;  // (the static array and a recorded request's slice may hold anything)
  }
}


}  // namespace rtams
