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

// ---- inner products on the matrix cores' double instructions.  v_mfma_f64_16x16x4 takes its four products one after the
// other, in order, each with a fused multiply-add (compared bit for bit with that chain over 51,200 sums of 96 products
// of widely spread sizes), so it IS the fixed arithmetic: 16 vectors against 16 centroids, one chunk of a row to an
// instruction.  (Sums of squared differences are no such product.)  The instruction does 16 multiply-adds a clock and
// SIMD, what the vector unit does too; what the kernel above loses is that every one of its multiply-adds takes a
// coordinate out of LDS, the same for all lanes, and here a word of LDS serves 16 of them.  What bounds it: the rate of
// the instruction where there are wavefronts for every SIMD (two tiles of 16 vectors against 8,192 centroids of 768
// dimensions add 12 us, 10.3 at 64 clocks an instruction), and the chain of one wavefront, d / 4 instructions, where there
// are not.  Choosing 16 of 8,192 lists, 768 dimensions, whole calls: 64 vectors 61 us through the kernel above, 49 here, 17
// vectors 62 and 38; 128 against 4,096 57 and 46; 64 against 8,192 lists of 1,536 dimensions 92 and 84, of 256 37 and 31.
// A wavefront has 16 centroids, which it reads from the transposed copy (a lane a float, 256 bytes of 16 centroids' chunk
// together), two sets of kDotSet chunks in turn, and 16 vectors, which the workgroup holds in LDS in the order of the
// lanes.  Two groups of vectors to a wavefront, which read the centroids half as often, or sets of 32 chunks are no faster.
typedef double DotAcc __attribute__((ext_vector_type(4)));
constexpr int kDotThreads = 256, kDotWaves = kDotThreads / kWave, kDotSet = 16;

__global__ __launch_bounds__(kDotThreads) void k_coarse_dots(Dev D, int64_t n, const float *__restrict__ Y,
                                                             double *__restrict__ scores, unsigned long long *cursor_to_clear,
                                                             uint32_t *__restrict__ zero, int zero_n) {
  extern __shared__ float s_dots[];  // [d4][64]: lane 16 g + v has coordinate g of the chunk, of vector v
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, d4 = D.d4;
  const int64_t v0 = (int64_t)blockIdx.x * 16;
  if (cursor_to_clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *cursor_to_clear = 0ull;
  if (zero) {
    const int nthreads = gridDim.x * gridDim.y * kDotThreads;
    for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * kDotThreads + threadIdx.x; i < zero_n; i += nthreads) zero[i] = 0u;
  }
  const int c = ((int)blockIdx.y * kDotWaves + wave) * 16 + (lane & 15);
  const float *col = D.centroids_t + (size_t)min(c, D.nlist - 1) * 4 + lane / 16;  // (past the end: dropped below)
  const size_t stride = (size_t)D.nlist * 4;
  float b0[kDotSet], b1[kDotSet];
  auto load_set = [&](float *b, int j0) {  // past the row's end its last chunk again
#pragma unroll
    for (int u = 0; u < kDotSet; ++u) b[u] = col[(size_t)min(j0 + u, d4 - 1) * stride];
    __builtin_amdgcn_sched_barrier(0);  // the loads go out here, not where they are used
  };
  load_set(b0, 0);
  for (int t = threadIdx.x; t < 16 * d4; t += kDotThreads) {
    const int v = t & 15, j = t >> 4;
    const int64_t row = v0 + v < n ? v0 + v : n - 1;
    const float4 y = reinterpret_cast<const float4 *>(Y)[(size_t)row * d4 + j];
    float *to = s_dots + (size_t)j * kWave + v;
    to[0] = y.x; to[16] = y.y; to[32] = y.z; to[48] = y.w;
  }
  __syncthreads();
  DotAcc acc = {0.0, 0.0, 0.0, 0.0};
  auto use_set = [&](const float *b, int j0) {  // a whole set
    float y[kDotSet];
#pragma unroll
    for (int u = 0; u < kDotSet; ++u) y[u] = s_dots[(size_t)(j0 + u) * kWave + lane];
#pragma unroll
    for (int u = 0; u < kDotSet; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)y[u], (double)b[u], acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto use_rest = [&](const float *b, int j0) {
#pragma unroll
    for (int u = 0; u < kDotSet; ++u) {
      if (j0 + u >= d4) break;  // uniform
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)s_dots[(size_t)(j0 + u) * kWave + lane], (double)b[u], acc, 0, 0, 0);
    }
  };
  int j = 0;
#pragma unroll 1
  for (; j + 2 * kDotSet <= d4; j += 2 * kDotSet) {
    load_set(b1, j + kDotSet);
    use_set(b0, j);
    load_set(b0, j + 2 * kDotSet);
    use_set(b1, j + kDotSet);
  }
  if (j < d4) {  // uniform
    if (j + kDotSet < d4) load_set(b1, j + kDotSet);
    use_rest(b0, j);
    if (j + kDotSet < d4) use_rest(b1, j + kDotSet);
  }
  if (c >= D.nlist) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t row = v0 + 4 * i + lane / 16;
    if (row < n) scores[(size_t)row * D.nlist + c] = acc[i];
  }
}

hipError_t allow_large_lds_dots() { return allow_lds(k_coarse_dots, 16 * 2048 * sizeof(float)); }  // (the widest vectors)

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

// Whether the scores of n vectors go to the matrix cores' double instructions.  Narrow vectors gain or lose nothing at any
// number of lists.  A wide vector's chain is longer there (64 clocks to four coordinates), which a batch that leaves the
// chip idle pays: from 2^17 pairs it is repaid, and from three eighths of that against 4,096 lists or more, where the kernel
// for vectors on their own, one to a workgroup, would read all the centroids for each.  Choosing 16 lists, us, the
// vector unit / here: 768 dimensions, 64 x 200 23 / 26, x 1,024 24 / 27, 128 x 1,024 30 / 30, 256 x 1,024 37 / 32, 8 x 4,096 33 /
// 30, 32 x 4,096 36 / 31; 1,536, 48 x 1,024 34 / 40, 128 x 1,024 47 / 46, 256 x 1,024 58 / 48, 17 x 4,096 61 / 48; 256, 64 x
// 1,024 18 / 19, 256 x 1,024 25 / 22, 8 x 4,096 21 / 22, 17 x 4,096 24 / 22; 128, 17 x
// 2,048 17 / 18; 96, 128 x 200 18 / 17, x 4,096 25 / 24.
static bool dots_pay(const Dev &D, int64_t n) {
  const int64_t pairs = n * D.nlist;
  return D.metric != 0 && n >= 8 && D.nlist <= 1 << 20 &&
         (D.d <= 96 || pairs >= (int64_t)1 << 17 || (D.nlist >= 4096 && pairs >= 3 << 14));
}

void launch_coarse_scores(const Dev &D, int64_t n, const float *Y, double *scores,
                          unsigned long long *cursor_to_clear, uint32_t *zero, int zero_n, hipStream_t s) {
  if (dots_pay(D, n)) {
    const dim3 grid((unsigned)((n + 15) / 16), (unsigned)((D.nlist + 16 * kDotWaves - 1) / (16 * kDotWaves)));
    hipLaunchKernelGGL(k_coarse_dots, grid, dim3(kDotThreads), (size_t)16 * D.d * sizeof(float), s, D, n, Y, scores,
                       cursor_to_clear, zero, zero_n);
    return;
  }
  int splits = coarse_splits(D, n, 0);
  launch_coarse<false>(D, n, Y, splits, scores, nullptr, nullptr, cursor_to_clear, zero, zero_n, s);
}

void launch_coarse_argmin(const Dev &D, int64_t n, const float *Y, int splits, double *pscore,
                          int32_t *pidx, hipStream_t s) {
  launch_coarse<true>(D, n, Y, splits, nullptr, pscore, pidx, nullptr, nullptr, 0, s);
}

}  // namespace rtams
