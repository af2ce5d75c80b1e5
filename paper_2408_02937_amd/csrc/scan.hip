// The list scan of flat lists: exact scores of every query against every vector of its probed lists.
#include "scan_item.h"

namespace rtams {

// The hardware's workgroup dispatcher is the work queue (a new workgroup starts
// wherever room frees up).  A workgroup is four wavefronts that take four
// consecutive work items, one each, and work on their own: own slice of LDS, no
// barrier.  Consecutive items are mostly the tiles of one segment, or the next
// segment of the same list.  Hardware hands consecutive workgroup ids to the 8
// XCDs in turn, so workgroup i runs on XCD i % 8 and takes items 4 (i / 8) ..
// 4 (i / 8) + 3 of that XCD's range of items (a contiguous range of lists).
// Wavefronts past the end of their range leave at once.

template <int METRIC, int ST, int G, int P>
__global__ __launch_bounds__(kScanWaves * kWave) void k_scan(Dev D, int max_nprobe,
                                                             const float *__restrict__ Q, SearchScratch S) {
  extern __shared__ float4 qs_all[];  // [wavefronts][kScanTileQueries][d / 4]
  const ScanQueues *Qs = S.queues;
  const uint32_t x = blockIdx.x % kXcds;
  const uint32_t wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
  const uint32_t item = Qs->begin[x] + (blockIdx.x / kXcds) * waves + wave;
  if (item >= Qs->begin[x + 1]) return;
  const uint32_t seg = Qs->seg_groups;
  if (seg == 0) return;
  float4 *qs = qs_all + (size_t)wave * kScanTileQueries * D.d4;
  const uint4 desc = S.tile_desc[item];
  const int list = __builtin_amdgcn_readfirstlane((int)desc.x);
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.y);
  const uint32_t pairs = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.z);
  const uint32_t g_begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.w) * seg;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t pk = lane < pairs ? S.grouped[first + lane] : 0u;  // the lane's pair
  switch (pairs) {
    case 0: break;
    case 1: scan_item<METRIC, 1, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 2: scan_item<METRIC, 2, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 3: scan_item<METRIC, 3, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 4: scan_item<METRIC, 4, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 5: scan_item<METRIC, 5, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 6: scan_item<METRIC, 6, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    case 7: scan_item<METRIC, 7, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
    default: scan_item<METRIC, 8, ST, G, P>(D, S, Q, max_nprobe, list, pk, g_begin, seg, qs); break;
  }
}


void launch_scan(const Dev &D, int64_t nq, int nprobe, int max_nprobe, const float *Q, int item_budget,
                 const SearchScratch &S, hipStream_t s) {
  if (nq <= 0) return;
  if (D.pq_m > 0) {
    launch_pq_scan(D, nq, nprobe, max_nprobe, item_budget, S, s);
    return;
  }
  const ScanShape sh = scan_shape(D, item_budget);
  if (D.scan_halves) {
    launch_scan_halves(D, sh, max_nprobe, S, s);
    return;
  }
  if (sh.mm) {
    launch_scan_mm(D, sh, max_nprobe, Q, S, s);
    return;
  }
  typedef void (*Kernel)(Dev, int, const float *, SearchScratch);
  static const Kernel pairs[2][3] = {{k_scan<0, 0, 2, 2>, k_scan<0, 1, 2, 2>, k_scan<0, 2, 2, 2>},
                                     {k_scan<1, 0, 2, 2>, k_scan<1, 1, 2, 2>, k_scan<1, 2, 2, 2>}};
  static const Kernel singles[2][3] = {{k_scan<0, 0, 1, 4>, k_scan<0, 1, 1, 4>, k_scan<0, 2, 1, 4>},
                                       {k_scan<1, 0, 1, 4>, k_scan<1, 1, 1, 4>, k_scan<1, 2, 1, 4>}};
  static const Kernel deep_singles[2] = {k_scan<0, 0, 1, 8>, k_scan<1, 0, 1, 8>};
  const Kernel kernel = sh.seg_base == 2 ? pairs[D.metric][D.storage]
                        : D.storage == 0 && D.vchunks % 16 == 0 ? deep_singles[D.metric] : singles[D.metric][D.storage];
  hipLaunchKernelGGL(kernel, dim3((unsigned)sh.grid), dim3((unsigned)sh.threads), sh.lds, s, D, max_nprobe, Q, S);
}

}  // namespace rtams
