// Probe selection and the per-query plan of a search request.
// (Paper, introduction: a query is compared with the lists of the clusters nearest to it only.)
#include "probe_plan.h"

namespace rtams {

// Workgroup of the probe selection: 256 threads, or 1024 where a query has thousands of centroids to
// go through (every pass of the selection reads them all).
constexpr int kSelThreads = 256, kSelThreadsMany = 1024, kSelManyFrom = 4096;

template <bool FROM_APPROX, int MINE>
__global__ __launch_bounds__(kSelThreadsMany) void k_probe_plan(Dev D, int64_t nq, int nprobe, int max_nprobe,
                                                            SearchScratch S, const float *__restrict__ Q,
                                                            int32_t *probe_out) {
  __shared__ ProbeShared<FROM_APPROX> sh;
  probe_plan<FROM_APPROX, MINE, false>(D, nq, (int)blockIdx.x, nprobe, max_nprobe, S, Q, probe_out, sh);
}

void launch_probe_plan(const Dev &D, int64_t nq, int nprobe, int max_nprobe, const SearchScratch &S,
                       const float *Q, bool from_approx, int32_t *probe_out, hipStream_t s) {
  if (nq <= 0) return;
  const unsigned threads = D.nlist >= kSelManyFrom ? kSelThreadsMany : kSelThreads;
  typedef void (*Kernel)(Dev, int64_t, int, int, SearchScratch, const float *, int32_t *);
  static const Kernel kernels[2][4] = {
      {k_probe_plan<false, 4>, k_probe_plan<false, 8>, k_probe_plan<false, 16>, k_probe_plan<false, 0>},
      {k_probe_plan<true, 4>, k_probe_plan<true, 8>, k_probe_plan<true, 16>, k_probe_plan<true, 0>}};
  const int per = (int)((D.nlist + threads - 1) / threads);  // scores of a row to a thread
  hipLaunchKernelGGL(kernels[from_approx ? 1 : 0][per <= 4 ? 0 : per <= 8 ? 1 : per <= 16 ? 2 : 3], dim3((unsigned)nq),
                     dim3(threads), 0, s, D, nq, nprobe, max_nprobe, S, Q, probe_out);
}

}  // namespace rtams
