// Coarse quantizer: score of every (vector, centroid) pair in the one fixed
// arithmetic that decides list membership and probe choice (IEEE double, one
// fused multiply-add per dimension, dimensions in ascending order), so that the
// integer decisions are reproducible bit for bit.  Insertion algorithm of the
// paper, step "k <- min(c, y_i)", and the first stage of search.
#include "coarse_exact.h"

namespace rtams {

// vectors per workgroup: their coordinates sit in LDS as doubles, 48 KiB at most (the workgroup has 3 KiB of its own)
int coarse_vt(int d) { return d <= 768 ? 8 : d <= 1536 ? 4 : 2; }
// ... and fewer for a small batch: every slot of a tile costs a full chain of fp64 operations per
// centroid whether a vector sits in it or not, and a batch of a few tiles leaves most of the chip
// idle (one workgroup per tile and centroid split).  The largest tile that still yields a
// workgroup per compute unit, else single vectors.
// Every multiply-add takes one coordinate of a vector out of LDS, the same for the whole wavefront,
// and with eight vectors to a thread the four wavefronts of a CU ask LDS for more than it returns
// (measured: 64 x 8,192 x 768 in 65 us, 15 % of the double-precision rate).  So where that rule picks
// eight or four vectors and there are 512 centroids or more, a thread takes half as many vectors
// against TWO centroids: the same number of chains per thread and of workgroups, half the reads of
// LDS per multiply-add (47 us for that batch).
struct CoarseShape {
  int vt;  // vectors of a workgroup's tile
  int nc;  // centroids a thread takes at a time
};
static CoarseShape coarse_shape(const Dev &D, int64_t n) {
  const int64_t max_s = (D.nlist + kCoarseThreads - 1) / kCoarseThreads;
  for (int vt = coarse_vt(D.d); vt > 1; vt /= 2)
    if ((n + vt - 1) / vt * max_s >= 256) {
      if (vt >= 4 && D.nlist >= 2 * kCoarseThreads) return {vt / 2, 2};
      return {vt, 1};
    }
  return {1, 1};
}

int coarse_vectors(const Dev &D, int64_t n) { return coarse_shape(D, n).vt; }

// How many workgroups share the centroids of one vector tile, so that a small
// batch still spreads over the chip.
int coarse_splits(const Dev &D, int64_t n, size_t part_cap) {
  const CoarseShape sh = coarse_shape(D, n);
  int64_t tiles = (n + sh.vt - 1) / sh.vt;
  int max_s = (D.nlist + sh.nc * kCoarseThreads - 1) / (sh.nc * kCoarseThreads);
  int64_t want = (1024 + tiles - 1) / tiles;
  int64_t s = want < 1 ? 1 : want;
  if (s > max_s) s = max_s;
  if (part_cap && (size_t)(s * n) > part_cap) s = (int64_t)(part_cap / (size_t)n);
  if (s < 1) s = 1;
  return (int)s;
}

template <int METRIC, int VT, int NC, bool ARGMIN>
__global__ __launch_bounds__(kCoarseThreads) void k_coarse(
    Dev D, int64_t n, const float *__restrict__ Y, int splits, double *__restrict__ scores,
    double *__restrict__ pscore, int32_t *__restrict__ pidx, unsigned long long *cursor_to_clear,
    uint32_t *__restrict__ zero, int zero_n) {
  coarse_tile<METRIC, VT, NC, ARGMIN, false, kCoarseThreads>(D, n, Y, splits, scores, pscore, pidx, cursor_to_clear, zero, zero_n);
}

// once per set_centroids: the transposed copy the kernel above streams
__global__ __launch_bounds__(256) void k_centroid_transpose(Dev D) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)D.nlist * D.d4) return;
  const int j = (int)(t / D.nlist), c = (int)(t % D.nlist);  // consecutive threads write consecutive 16 bytes
  reinterpret_cast<float4 *>(D.centroids_t)[t] = reinterpret_cast<const float4 *>(D.centroids)[(size_t)c * D.d4 + j];
}

void launch_centroid_transpose(const Dev &D, hipStream_t s) {
  const int64_t items = (int64_t)D.nlist * D.d4;
  hipLaunchKernelGGL(k_centroid_transpose, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, D);
}

template <bool ARGMIN>
static void launch_coarse(const Dev &D, int64_t n, const float *Y, int splits, double *scores,
                          double *pscore, int32_t *pidx, unsigned long long *cursor, uint32_t *zero,
                          int zero_n, hipStream_t s) {
  if (n <= 0) return;
  const CoarseShape sh = coarse_shape(D, n);
  const int vt = sh.vt;
  dim3 grid((unsigned)((n + vt - 1) / vt), (unsigned)splits);
  size_t lds = (size_t)vt * D.d * sizeof(double);
#define RTAMS_GO(M, V, N_) \
  hipLaunchKernelGGL((k_coarse<M, V, N_, ARGMIN>), grid, dim3(kCoarseThreads), lds, s, D, n, Y, splits, \
                     scores, pscore, pidx, cursor, zero, zero_n)
  if (D.metric == 0) {
    if (vt == 8) RTAMS_GO(0, 8, 1); else if (vt == 4 && sh.nc == 2) RTAMS_GO(0, 4, 2); else if (vt == 4) RTAMS_GO(0, 4, 1);
    else if (vt == 2 && sh.nc == 2) RTAMS_GO(0, 2, 2); else if (vt == 2) RTAMS_GO(0, 2, 1); else RTAMS_GO(0, 1, 1);
  } else {
    if (vt == 8) RTAMS_GO(1, 8, 1); else if (vt == 4 && sh.nc == 2) RTAMS_GO(1, 4, 2); else if (vt == 4) RTAMS_GO(1, 4, 1);
    else if (vt == 2 && sh.nc == 2) RTAMS_GO(1, 2, 2); else if (vt == 2) RTAMS_GO(1, 2, 1); else RTAMS_GO(1, 1, 1);
  }
#undef RTAMS_GO
}

void launch_coarse_scores(const Dev &D, int64_t n, const float *Y, double *scores,
                          unsigned long long *cursor_to_clear, uint32_t *zero, int zero_n, hipStream_t s) {
  int splits = coarse_splits(D, n, 0);
  launch_coarse<false>(D, n, Y, splits, scores, nullptr, nullptr, cursor_to_clear, zero, zero_n, s);
}

void launch_coarse_argmin(const Dev &D, int64_t n, const float *Y, int splits, double *pscore,
                          int32_t *pidx, hipStream_t s) {
  launch_coarse<true>(D, n, Y, splits, nullptr, pscore, pidx, nullptr, nullptr, 0, s);
}

}  // namespace rtams
