// A small request over flat lists in three launches instead of five: coarse scores, probes and bound in one kernel, a scan
// that finds its own work, the selection.
//
// What bounds such a request is the chain of its launches, each with a start and an end of two microseconds and a few trips
// to memory before it has what the one before it left behind, and the plan: pairs counted and grouped by list, work items
// cut and shared out by one workgroup, which a request whose pairs hardly share a list does not get back.  Here the last
// workgroup of a query's coarse scores goes on with its probes and its bound, and the wavefronts of the scan take the
// groups of the query's lists in turn from the lengths alone.
// 10 queries x 8 probes over 64 lists, 10,000 x 32 floats: 31.6 us back to back where the five launches took 42.7; one
// query x 32 probes over 1,024 lists, 1 M x 128: 45.7 and 47.3.  Above kSmallBytes the scan's own time hides the
// plan, and what several queries read of one list is read once.  Wide vectors: small_request().
#include "bound.h"
#include "coarse_exact.h"
#include "probe_plan.h"
#include "scan_item.h"

namespace rtams {

constexpr int kSmallThreads = 512;  // eight wavefronts: the bound's sample of 512 vectors in one turn
// (With three kernels' worth of code in one, k_small_front spills 28 to 53 scalar registers to lanes of vector registers, 169
// of them.  At one query it takes 19 us where coarse scores, probes and bound took 4.6, 6.8 and 8.5: what is saved is launches.)

template <int METRIC, int MINE>
__global__ __launch_bounds__(kSmallThreads) void k_small_front(Dev D, int64_t nq, int nprobe, int max_nprobe, int k,
                                                               const float *__restrict__ Q, int splits, SearchScratch S) {
  // (the probes' keys, then the bound's query and sample)
  __shared__ __attribute__((aligned(16))) unsigned char s_raw[kBoundLdsBytes];
  static_assert(sizeof(ProbeShared<false>) <= kBoundLdsBytes, "the probes share the bound's LDS");
  __shared__ uint32_t s_last;
  const int q = blockIdx.x;
  coarse_tile<METRIC, 1, 1, false, true, kSmallThreads>(D, nq, Q, splits, S.scores, nullptr, nullptr, nullptr, nullptr, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's scores are out ...
  __syncthreads();                                  // ... and so are everybody's before the workgroup counts itself off
  if (splits > 1) {  // uniform
    if (threadIdx.x == 0) {
      s_last = atomicAdd(&S.done_count[q], 1u) + 1u == (uint32_t)splits;
      if (s_last) S.done_count[q] = 0u;  // for the next request
    }
    __syncthreads();
    if (!s_last) return;  // uniform: the last one goes on
  }
  probe_plan<false, MINE, true>(D, nq, q, nprobe, max_nprobe, S, Q, nullptr, *reinterpret_cast<ProbeShared<false> *>(s_raw));
  __syncthreads();  // the plan is read below by other threads, and its LDS is used again
  sample_bound<false, false>(D, q, nprobe, max_nprobe, k, Q, S, s_raw, 0u, 1u);
}

// Workgroup `part` of the `parts` of query q: its wavefronts take every (parts x wavefronts)-th unit of G groups of the
// query's lists, counted list after list.  At most 64 probes, a lane to each.
template <int METRIC, int ST, int G, int P>
__global__ __launch_bounds__(kScanWaves * kWave) void k_scan_small(Dev D, int nprobe, int max_nprobe, int parts,
                                                                   const float *__restrict__ Q, SearchScratch S) {
  extern __shared__ float4 qs_small[];  // [wavefronts][d / 4]
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave), waves = blockDim.x / kWave;
  const uint32_t q = blockIdx.x / (uint32_t)parts, part = blockIdx.x % (uint32_t)parts;
  float4 *qs = qs_small + (size_t)wave * D.d4;
  const size_t o = (size_t)q * max_nprobe + min(lane, nprobe - 1);
  const int my_list = S.probe_list[o];
  const uint32_t my_len = S.probe_len[o];
  const uint32_t have = D.nblk[my_list] * (uint32_t)D.groups_per_block;  // never past the list's chain
  const uint32_t units = lane < nprobe ? (min((my_len + kWave - 1) / kWave, have) + G - 1) / G : 0u;
  const uint32_t upto = wave_running_sum(units), total = last_lane(upto);
  const uint32_t first = units ? upto - units : ~0u;  // the lane's probe starts at this unit
  for (uint32_t u = part * waves + wave; u < total; u += (uint32_t)parts * waves) {  // uniform over the wavefront
    const int p = 63 - __clzll((long long)__ballot(first <= u));  // the last probe that starts at or before u
    const uint32_t g = (u - (uint32_t)__builtin_amdgcn_readlane((int)first, p)) * G;
    scan_item<METRIC, 1, ST, G, P>(D, S, Q, max_nprobe, __builtin_amdgcn_readlane(my_list, p), q << 10 | (uint32_t)p, g, G, qs);
  }
}

bool small_request(const Dev &D, int64_t nq, int nprobe, int64_t avg_len, int64_t longest) {
  if (D.pq_m > 0 || D.scan_mfma || D.nlist < 32 || D.nlist > 4096 || nprobe > kWave || coarse_vectors(D, nq) != 1) return false;
  // every query reads its lists for itself
  if ((double)nq * (double)(nprobe * avg_len + longest) * D.vchunks * 16.0 > kSmallBytes) return false;
  // Half as many workgroups as in a planned request read the centroids here, and one the sample of a query, which a planned
  // request of few queries shares between four: with wide vectors that takes longer than two launches, unless many pairs
  // make the plan long, many queries fill the chip (53 x 3 probes, 438 short lists x 776: 54 us, planned 61), or a planned
  // request has one workgroup for the centroids as well, up to 256 of them.  Small / planned, the middle and the largest of
  // 5 to 60 requests each of 1 to 32 queries x 8 to 64 probes over 64 to 4,096 lists of up to 1,500 vectors, up to 32 MB:
  //  d 32 0.81 to 0.90, 1.01; d 128 0.81 to 0.95, 1.02; d 256 0.86 to 0.97, 1.00; d 512 without a bound 0.80 to 0.94, 1.00,
  //    with one and long lists of floats 1.01, 1.06, of halves and bytes 1.00, 1.04
  //  long lists, d 768: floats 1.12, halves and bytes 0.93 to 1.00, 1.00, with a bound 1.02, 1.05
  //  short lists, floats: d 768 0.88 to 0.98, 1.04, d 1024 0.91 to 1.03, 1.09, d 1536 0.97 to 1.11, 1.22, of these from 400
  //    pairs 0.82 to 0.99, 1.02; halves and bytes: d 1024 0.80 to 0.95, 1.02, d 1536 0.81 to 1.03, 1.18, from 100 pairs 0.48
  //    to 0.83, 0.83, d 2048 from 128 pairs 1.04 to 1.07, 1.12, from 256 0.51 to 0.82, 1.05
  const bool short_lists = avg_len / kWave + 1 <= kSingleList;  // a sample is a few groups of each, shared or not
  const bool narrow = D.storage != 0;
  const int wide = short_lists ? (narrow ? 1024 : 768) : (narrow ? 768 : 512);
  if (D.d > wide && D.nlist > 256 && !(short_lists && (nq >= 16 || nq * nprobe >= (narrow ? 100 : 400) * (D.d > 1536 ? 2 : 1)))) return false;
  const int64_t no_bound_below = D.metric == 0 ? 4096 : 32 * (int64_t)D.d > 4096 ? 32 * (int64_t)D.d : 4096;
  return short_lists || nprobe * avg_len <= no_bound_below || (D.vchunks < 96 && D.d <= 512);
}

void launch_small_front(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int k, const float *Q, const SearchScratch &S,
                        hipStream_t s) {
  const int splits = (D.nlist + kSmallThreads - 1) / kSmallThreads;  // a centroid to a thread
  typedef void (*Kernel)(Dev, int64_t, int, int, int, const float *, int, SearchScratch);
  static const Kernel kernels[2][3] = {{k_small_front<0, 2>, k_small_front<0, 4>, k_small_front<0, 8>},
                                       {k_small_front<1, 2>, k_small_front<1, 4>, k_small_front<1, 8>}};
  hipLaunchKernelGGL(kernels[D.metric][splits <= 2 ? 0 : splits <= 4 ? 1 : 2], dim3((unsigned)nq, (unsigned)splits),
                     dim3(kSmallThreads), (size_t)D.d * sizeof(double), s, D, nq, nprobe, max_nprobe, k, Q, splits, S);
}

void launch_scan_small(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int64_t units, const float *Q,
                       const SearchScratch &S, hipStream_t s) {
  // a unit to a wavefront while the chip has room for them, by what a query's lists may come to
  int64_t parts = (units + kScanWaves - 1) / kScanWaves;
  const int64_t most = (1024 + nq - 1) / nq;
  parts = parts < 1 ? 1 : parts > most ? most : parts;
  typedef void (*Kernel)(Dev, int, int, int, const float *, SearchScratch);
  static const Kernel pairs[2][3] = {{k_scan_small<0, 0, 2, 2>, k_scan_small<0, 1, 2, 2>, k_scan_small<0, 2, 2, 2>},
                                     {k_scan_small<1, 0, 2, 2>, k_scan_small<1, 1, 2, 2>, k_scan_small<1, 2, 2, 2>}};
  static const Kernel singles[2][3] = {{k_scan_small<0, 0, 1, 4>, k_scan_small<0, 1, 1, 4>, k_scan_small<0, 2, 1, 4>},
                                       {k_scan_small<1, 0, 1, 4>, k_scan_small<1, 1, 1, 4>, k_scan_small<1, 2, 1, 4>}};
  static const Kernel deep_singles[2] = {k_scan_small<0, 0, 1, 8>, k_scan_small<1, 0, 1, 8>};
  const Kernel kernel = !D.scan_single ? pairs[D.metric][D.storage]
                        : D.storage == 0 && D.vchunks % 16 == 0 ? deep_singles[D.metric] : singles[D.metric][D.storage];
  hipLaunchKernelGGL(kernel, dim3((unsigned)(nq * parts)),
                     dim3(kScanWaves * kWave), (size_t)kScanWaves * D.d * sizeof(float), s, D, nprobe, max_nprobe, (int)parts, Q, S);
}

}  // namespace rtams
