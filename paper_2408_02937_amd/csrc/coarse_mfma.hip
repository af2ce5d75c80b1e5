// Coarse quantizer as a dense contraction on the matrix cores, used when a
// batch is large enough for that to pay (bulk loads, big insertion batches,
// query batches against many centroids): approximate scores of every (vector,
// centroid) pair.
//
// The approximate scores only FILTER.  Which list a vector joins and which
// lists a query probes are decided by the fixed double-precision arithmetic of
// coarse.hip on the few centroids the filter cannot tell apart (refinement
// kernels below and in probe.hip), so the decisions stay bit-exact.
//
// One product of halves is enough for that.  Let mu be the mean of the centroids,
// c' = c - mu, y' = y - mu (each a rounded fp32 subtraction), and h(x) the value of
// x as a half under a power-of-two scale (one for all centroids, one per vector;
// what would be a subnormal half becomes zero).  Up to a term that is the same for
// every centroid the score of (y, c) is, smaller is better,
//   b_c - g <y', c'>,   g = 2, b_c = |c'|^2 (L2)      g = 1, b_c = -<mu, c'> (IP)
// and what the kernel computes is b_c - g <h(y'), h(c')>: products of two halves are
// exact in fp32 and are accumulated in fp32.  With r(x) = |x - h(x)|, which is
// COMPUTED (per vector, and the largest over the centroids) and not assumed, n(x) = |x|:
//   |approx - exact| <= E = g (r(y') n_c + (n(y') + r(y')) r_c + d 2^-23 n_h(y) n_h(c))
//                          + 2^-22 (max |b_c| + g n(y') n_c + m)
// the first two terms by Cauchy and Schwarz, the third for d additions in any order
// (2^-23: an addition may round either way), the last for the roundings of b_c, of the
// final combination and of the two subtractions (m = (n(y') + n_c)^2 for L2,
// n_c (|mu| + 2 n(y')) for IP).  If t is the smallest approximate score of a row, the
// exact winner lies among the centroids with approx <= t + 2 E.  Byte-valued data is
// exact in a half; for real-valued data r is about 2^-12.3 of the norm, and one or two
// centroids of thousands lie within the band.  Without the centring the band would
// grow with the distance of the data from the origin, which decides nothing.
// (What this replaces: three products of bf16 pairs, a band of 2^-14 of the squared
// norms, three times the matrix instructions and twice the operand bytes: 324 us for
// 13,107 x 16,384 x 256, 728 us for 21,845 x 8,192 x 768.)
// Vectors whose band is not finite (infinities, overflow, centroids that are not finite or
// too large) are scored exactly against every centroid: their scale is zero, so that every
// approximate score is the centroid's bias, a finite number, and none drops out.  A vector
// with a NaN compares with nothing and goes to the first list, as it does in the exact
// arithmetic.
//
// For a search the whole score matrix is written (probe selection needs the
// nprobe-th smallest of a row).  For an assignment it is not: each workgroup
// reduces its tile on the spot to, per row, the tile's smallest score and the (up to
// kTileCands) columns within the band of it; the refinement reads those few bytes
// per (row, tile) instead of the matrix, twice.
#include <type_traits>
#include "rtams_launch.h"

namespace rtams {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

constexpr int kMfmaThreads = 256;  // 4 wavefronts: 2 (vectors) x 2 (centroids)
constexpr int kTileM = 128;        // vectors of a tile: 64 to a wavefront
constexpr int kTileK = 32;         // coordinates per step
constexpr int kBuffers = 3;        // steps whose operands have room in LDS
constexpr int kXcds = 8;  // workgroups go to the chip's 8 dies (each with its own L2) in turn

// Operands in memory lie as the tiles are read: blocks of 16 rows x 32 coordinates, 1 KiB each, the steps of a
// block of rows one after the other.  Inside a block row r has four 16-byte places, and group g of 8 coordinates
// is at place g ^ place_swap(r): the 8 rows that neighbouring lanes read from LDS then cover 32 banks once, and the
// 16 rows of a quarter of a wavefront all 64, with no padding, and a copy of a block to LDS is 1 KiB in order.
__device__ inline int place_swap(int row) { return ((row >> 1) & 2) | (((row >> 1) ^ (row >> 3)) & 1); }
__device__ inline size_t operand_at(int64_t row, int g, int steps) {
  return ((size_t)(row >> 4) * steps + (g >> 2)) * 64 + (size_t)(row & 15) * 4 + ((g & 3) ^ place_swap((int)row & 15));
}

__device__ inline uint32_t pack_halves_flushed(float a, float b) {  // nearest even; subnormal halves become zero
  halfx2 p;
  p[0] = (_Float16)(fabsf(a) < 6.103515625e-05f ? 0.f : a);
  p[1] = (_Float16)(fabsf(b) < 6.103515625e-05f ? 0.f : b);
  return __builtin_bit_cast(uint32_t, p);
}
// power of two that brings `top` (the largest magnitude of a row) into 2^13 .. 2^14, as far as a float can
__device__ inline float half_scale(float top) {
  if (!(top > 0.f) || !(top < __builtin_inff())) return 1.f;
  const int e = (int)((__float_as_uint(top) >> 23) & 255u) - 127;  // (a subnormal float counts as 2^-127)
  int s = 13 - e;
  s = s > 100 ? 100 : s < -114 ? -114 : s;
  return __uint_as_float((uint32_t)(s + 127) << 23);
}
// 8 scaled coordinates -> 8 halves; adds their squares and the squares of what the halves leave out
__device__ inline u32x4 halves_of(const float *x, float &nsq, float &rsq) {
  u32x4 out;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = x[2 * j], b = x[2 * j + 1];
    const uint32_t packed = pack_halves_flushed(a, b);
    const halfx2 h = __builtin_bit_cast(halfx2, packed);
    out[j] = packed;
    const float ra = a - (float)h[0], rb = b - (float)h[1];  // exact
    nsq = fmaf(a, a, nsq); nsq = fmaf(b, b, nsq);
    rsq = fmaf(ra, ra, rsq); rsq = fmaf(rb, rb, rsq);
  }
  return out;
}
// coordinates 8 g .. 8 g + 7 of a row less the mean; zero past d (the row's last chunk is asked for there: a branch
// around every load would keep the loads of a row apart)
__device__ inline void centred_group(const Dev &D, const float *row, int g, float *x) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int j = g * 8 + q * 4, at = min(j, D.d - 4);
    const float4 u = *reinterpret_cast<const float4 *>(row + at), m = *reinterpret_cast<const float4 *>(D.cmean + at);
    x[4 * q] = j < D.d ? u.x - m.x : 0.f; x[4 * q + 1] = j < D.d ? u.y - m.y : 0.f;
    x[4 * q + 2] = j < D.d ? u.z - m.z : 0.f; x[4 * q + 3] = j < D.d ? u.w - m.w : 0.f;
  }
}
__device__ inline float group_top(const float *x) {
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) t = fmaxf(t, fabsf(x[j]));
  return t;
}

// ---- once per set_centroids, behind the transposed copy: the mean of the centroids (a workgroup per chunk of 4
// coordinates), their largest centred magnitude, then bias, halves and the largest norms
__global__ __launch_bounds__(256) void k_centroid_mean(Dev D) {
  __shared__ double s_sum[4][4];
  const int j = blockIdx.x, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (j == 0 && threadIdx.x == 0) {
    D.ctrl->cen = CentroidStats{};
    D.ctrl->half_top = 0u;
    D.ctrl->half_inexact = 0u;
  }
  const float4 *col = reinterpret_cast<const float4 *>(D.centroids_t) + (size_t)j * D.nlist;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c = threadIdx.x; c < D.nlist; c += 256) {
    const float4 v = col[c];
    a[0] += (double)v.x; a[1] += (double)v.y; a[2] += (double)v.z; a[3] += (double)v.w;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    for (int o = kWave / 2; o > 0; o >>= 1) a[u] += __shfl_xor(a[u], o);
    if (lane == 0) s_sum[u][wave] = a[u];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const double *p = s_sum[threadIdx.x];
    const float m = (float)((p[0] + p[1] + p[2] + p[3]) / (double)D.nlist);
    // (a centroid that is not finite has no share in the mean, or it would take every vector with it)
    D.cmean[4 * j + threadIdx.x] = fabsf(m) < __builtin_inff() ? m : 0.f;
  }
}

// Largest of a value per wavefront over the workgroup, into a word of float bits (non-negative floats order like their
// bits).  Atomics on one word follow each other at about 12 ns, and that is what bounds both kernels below: one per
// centroid took 0.2 ms for 16,384 of them, one per workgroup of 4 wavefronts and word 18 us of the 33 and 38 that 8,192 x
// 768 took; 13 and 27 now.  So workgroups are the largest there are, and a value that cannot change the word stays out of the line: zero,
// or no larger than what a look at the word finds there (it only grows; an old value costs an atomic, no more).
constexpr int kTopThreads = 1024, kTopWaves = kTopThreads / kWave;
__device__ inline void wg_atomic_max(float v, float *lds, uint32_t *word) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  __syncthreads();
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kTopWaves; ++w) v = fmaxf(v, lds[w]);
    const uint32_t bits = __float_as_uint(v);
    if (bits > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(word, bits);
  }
}

// a wavefront per centroid, in turns; four chunks of a row to a lane asked for at once (past the row's end its last
// chunk again, which changes no maximum)
__global__ __launch_bounds__(kTopThreads) void k_centroid_top(Dev D) {
  __shared__ float s_max[kTopWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const float4 *mean = reinterpret_cast<const float4 *>(D.cmean);
  float top = 0.f, bad = 0.f, whole = 0.f;
  auto look = [&](float x, float m) {
    const float v = fabsf(x - m);
    if (!(v < 1e17f) || !(fabsf(m) < 1e17f)) bad = 1.f;  // (squares and products of these, summed, stay finite)
    top = fmaxf(top, v);
    whole = fmaxf(whole, fabsf(x) < __builtin_inff() ? fabsf(x) : 0.f);
  };
  for (int c = blockIdx.x * kTopWaves + threadIdx.x / kWave; c < D.nlist; c += gridDim.x * kTopWaves) {
    const float4 *row = reinterpret_cast<const float4 *>(D.centroids + (size_t)c * D.d);
    for (int j0 = 0; j0 < D.d4; j0 += 4 * kWave) {
      float4 x[4], m[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = min(j0 + u * kWave + lane, D.d4 - 1);
        x[u] = row[j];
        m[u] = mean[j];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        look(x[u].x, m[u].x); look(x[u].y, m[u].y); look(x[u].z, m[u].z); look(x[u].w, m[u].w);
      }
    }
  }
  wg_atomic_max(top, s_max, &D.ctrl->cen.top_bits);
  wg_atomic_max(bad, s_max, &D.ctrl->cen.bad);
  wg_atomic_max(whole, s_max, &D.ctrl->half_top);
}

__global__ __launch_bounds__(kTopThreads) void k_centroid_halves(Dev D) {
  __shared__ float s_max[kTopWaves];
  const int lane = threadIdx.x & (kWave - 1);
  CentroidStats &st = D.ctrl->cen;
  const float scale = half_scale(__uint_as_float(st.top_bits));
  const bool bad = st.bad != 0u;  // no centroid is told apart by the filter then
  float top_n = 0.f, top_r = 0.f, top_b = 0.f;
  for (int c = blockIdx.x * kTopWaves + threadIdx.x / kWave; c < D.nlist; c += gridDim.x * kTopWaves) {  // uniform over the wavefront
    const float *row = D.centroids + (size_t)c * D.d;
    float nsq = 0.f, rsq = 0.f;
    double bias = 0.0;
    for (int g = lane; g < D.dgroups; g += kWave) {
      float x[8];
      centred_group(D, row, g, x);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double m = g * 8 + j < D.d ? (double)D.cmean[g * 8 + j] : 0.0;
        bias = D.metric == 0 ? __builtin_fma((double)x[j], (double)x[j], bias) : __builtin_fma(-m, (double)x[j], bias);
        x[j] = bad ? 0.f : x[j] * scale;
      }
      D.chalf[operand_at(c, g, D.dgroups / 4)] = halves_of(x, nsq, rsq);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) { nsq += __shfl_xor(nsq, o); rsq += __shfl_xor(rsq, o); bias += __shfl_xor(bias, o); }
    const float b = bad ? 0.f : (float)bias;
    if (lane == 0) D.cbias[c] = b;
    top_n = fmaxf(top_n, sqrtf(nsq)); top_r = fmaxf(top_r, sqrtf(rsq)); top_b = fmaxf(top_b, fabsf(b));
  }
  wg_atomic_max(top_n, s_max, &st.norm_bits);
  wg_atomic_max(top_r, s_max, &st.res_bits);
  wg_atomic_max(top_b, s_max, &st.bias_bits);
  if (blockIdx.x == 0 && threadIdx.x < kWave) {
    double m = 0.0;
    for (int j = lane; j < D.d; j += kWave) m = __builtin_fma((double)D.cmean[j], (double)D.cmean[j], m);
    for (int o = kWave / 2; o > 0; o >>= 1) m += __shfl_xor(m, o);
    if (lane == 0) {
      st.mean_norm = (float)__builtin_sqrt(m);
      D.ctrl->half_scale = halves_scale_for(D.ctrl->half_top);
    }
  }
}

// ---- the vectors of a batch: halves, and per row what turns an accumulated product into a score (g over the two
// scales) and the band 2 E.  `lpr` lanes of a wavefront take a row (4 .. 64, a power of two), G groups of 8
// coordinates each, which stay in registers between the look for the largest one and the conversion.
template <int G>
__global__ __launch_bounds__(256) void k_half_rows(Dev D, int64_t n, const float *__restrict__ Y, int lpr,
                                                   u32x4 *__restrict__ half, RowMeta *__restrict__ meta) {
  const int lane = threadIdx.x & (kWave - 1), sub = lane & (lpr - 1);
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / lpr;
  const bool on = i < n;
  const float *row = Y + (on ? i : n - 1) * D.d;
  float x[G][8], top = 0.f;
#pragma unroll
  for (int t = 0; t < G; ++t) centred_group(D, row, sub + t * lpr, x[t]);  // groups past the row are past d: zero
#pragma unroll
  for (int t = 0; t < G; ++t) top = fmaxf(top, group_top(x[t]));
  for (int o = lpr / 2; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
  const float scale = half_scale(top);
  const bool bad = !(top < __builtin_inff());
  if (bad) {  // what is left of such a row are its NaNs (every comparison and select of this kernel is paid per coordinate)
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[t][j] = x[t][j] == x[t][j] ? 0.f : x[t][j];
  }
  float nsq = 0.f, rsq = 0.f;
#pragma unroll
  for (int t = 0; t < G; ++t) {
    const int g = sub + t * lpr;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[t][j] *= scale;
    const u32x4 h = halves_of(x[t], nsq, rsq);
    if (on && g < D.dgroups) half[operand_at(i, g, D.dgroups / 4)] = h;
  }
  for (int o = lpr / 2; o > 0; o >>= 1) { nsq += __shfl_xor(nsq, o); rsq += __shfl_xor(rsq, o); }
  if (!on || sub != 0) return;
  const CentroidStats &st = D.ctrl->cen;
  const float iy = 1.f / scale, ic = 1.f / half_scale(__uint_as_float(st.top_bits));  // powers of two: exact
  const float g = D.metric == 0 ? 2.f : 1.f;
  const float ny = sqrtf(nsq), ry = sqrtf(rsq), nc = __uint_as_float(st.norm_bits), rc = __uint_as_float(st.res_bits);
  float s = g * iy * ic;
  const float e = s * (ry * nc + (ny + ry) * rc + (float)D.d * 1.1920929e-7f * (ny + ry) * (nc + rc));
  const float uy = ny * iy, uc = nc * ic;  // the norms themselves
  const float m = D.metric == 0 ? (uy + uc) * (uy + uc) : uc * (st.mean_norm + 2.f * uy);
  float band = 2.f * (1.01f * e + 2.3841858e-7f * 1.01f * (__uint_as_float(st.bias_bits) + s * ny * nc + m)) * 1.01f;
  // nothing is told apart by the filter where the band says nothing: infinities, or numbers at the ends of the
  // float range (a NaN in the vector stays out: no comparison holds for it anywhere).  The lower end: the scale has to be
  // a normal float, and the hundredth by which the band is widened has to cover what the dozen operations of the band, the
  // bias and the score lose below the smallest normal float, 1.2e-38 each even if subnormals became zero.  Vectors and
  // centroids of norms down to 1e-14 stay above both; what lies below is scored exactly against every centroid.
  if (bad || st.bad != 0u || !(band > 1e-34f) || !(band < 1e37f) || !(s >= 1.17549435e-38f)) {
    band = __builtin_inff();
    s = 0.f;  // (the products may overflow, or the scale itself, which times a product of zero is a NaN)
  }
  meta[i] = RowMeta{s, band};
}

// ---- approximate scores of a tile of 128 vectors x 64 CA centroids; a wavefront has 64 vectors x 32 CA centroids.
// With CA = 4 a step of 32 coordinates is 16 matrix instructions of 32 clocks to a wavefront between two barriers.
// CA = 2 is for batches whose wide tiles would leave compute units without a workgroup.
// Three buffers in LDS: a step's operands are copied there straight from memory (no registers in between) two steps
// ahead of the multiplications, and the one barrier of a step waits for the copies of that step alone, the next
// step's stay on their way.  Two workgroups share a compute unit, and one's waits are the other's multiplications.
// What bounds it: inside the steps the matrix cores are busy 85 % of the clocks, and the chip lowers its clock to 1.6 to
// 1.7 GHz under them; the reduction of a tile (6 us of the 25 that a tile of 768 dimensions is on a compute unit)
// overlaps with the steps of the other workgroup (it keeps the masks of many comparisons at a time and spills 175 scalar
// registers to lanes of vector registers at CA = 4, 47 at CA = 2).  28,928 x 8,192 x 768 take 370 us, 980 TFLOP/s; 424 us with
// two buffers filled through registers a step ahead and a branch for every score in the reduction, 30 % of the LDS
// clocks bank conflicts (the places of a row's groups covered 32 banks, not 64).
template <int CA, bool MATRIX>
__global__ __launch_bounds__(kMfmaThreads, 2) void k_coarse_mfma(Dev D, int64_t n, const u32x4 *__restrict__ yhalf,
                                                              const RowMeta *__restrict__ meta,
                                                              float *__restrict__ approx, TileCands tc, int die_map,
                                                              unsigned long long *cursor_to_clear,
                                                              uint32_t *__restrict__ zero, int zero_n) {
  constexpr int kTileN = 64 * CA;
  constexpr int kUnitsY = kTileM * 4 / kMfmaThreads, kUnitsC = kTileN * 4 / kMfmaThreads;  // copies of 1 KiB a wavefront makes per step
  constexpr int kBuf = (kTileM + kTileN) * 4;  // 16-byte units of a buffer: the vectors', then the centroids'
  extern __shared__ u32x4 s_op[];              // kBuffers of them
  __shared__ float s_min[kTileM][2];
  __shared__ float s_cn[kTileN];  // bias of the tile's centroids
  __shared__ uint32_t s_cnt[kTileM];
  __shared__ __attribute__((aligned(16))) uint16_t s_kept[kTileM][kTileCands];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wv = wave & 1, wc = wave >> 1;  // wavefront's place in the 2 (vectors) x 2 (centroids) arrangement

  // per-request counters of the search plan start from zero (no memset node on the stream)
  if (cursor_to_clear && blockIdx.x == 0 && tid == 0) *cursor_to_clear = 0ull;
  if (zero) {
    const int nthreads = gridDim.x * kMfmaThreads;
    for (int i = blockIdx.x * kMfmaThreads + tid; i < zero_n; i += nthreads) zero[i] = 0u;
  }

  // Which tile: consecutive workgroups land on consecutive dies, so die x takes the column tiles
  // x, x + 8, ... and walks the row tiles with them: the centroids of its column tiles stay in
  // its L2 (1 MiB of 4 for 16,384 centroids of 256 dimensions) while the vectors stream through once.
  // (Few column tiles: they are dealt out in turn, so that every die has its share.)
  const int col_tiles = (D.nlist + kTileN - 1) / kTileN;
  int col_tile;
  int64_t row_tile;
  if (die_map) {
    const int per_die = (col_tiles + kXcds - 1) / kXcds;
    const int die = blockIdx.x % kXcds, turn = blockIdx.x / kXcds;
    col_tile = (turn % per_die) * kXcds + die;
    if (col_tile >= col_tiles) return;  // uniform
    row_tile = turn / per_die;
  } else {
    col_tile = blockIdx.x % col_tiles;
    row_tile = blockIdx.x / col_tiles;
  }
  const int64_t row0 = row_tile * kTileM;
  const int col0 = col_tile * kTileN;

  // (asked for in front of the copies, put into LDS behind the multiplications)
  const float bias = tid < kTileN && col0 + tid < D.nlist ? D.cbias[col0 + tid] : __builtin_inff();

  floatx16 acc[CA][2];
#pragma unroll
  for (int a = 0; a < CA; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  // Copies: a wavefront brings blocks of 16 rows, 1 KiB each.  Blocks past the last vector or centroid read the
  // last one, and rows of the last block past the end hold whatever the memory holds: the scores of both are dropped.
  const int steps = D.dgroups / 4;
  const u32x4 *src[kUnitsY + kUnitsC];  // the same for every lane
  {
    const int64_t last_y = (n - 1) >> 4;
    const int last_c = (D.nlist - 1) >> 4;
#pragma unroll
    for (int h = 0; h < kUnitsY; ++h) {
      const int64_t blk = (row0 >> 4) + wave + 4 * h;
      src[h] = yhalf + (size_t)(blk < last_y ? blk : last_y) * steps * 64;
    }
#pragma unroll
    for (int h = 0; h < kUnitsC; ++h) {
      const int blk = (col0 >> 4) + wave + 4 * h;
      src[kUnitsY + h] = D.chalf + (size_t)(blk < last_c ? blk : last_c) * steps * 64;
    }
  }
  const uint32_t lds0 = lds_address(s_op) + (uint32_t)wave * 1024u;
  const uint32_t lane_off = (uint32_t)lane * 16u;
  auto fetch = [&](int st) {  // asks for a step's operands; they lie in the step's buffer when the wavefront's count of loads says so
    const uint32_t to = lds0 + (uint32_t)(st % kBuffers) * (kBuf * 16u);
#pragma unroll
    for (int h = 0; h < kUnitsY + kUnitsC; ++h)
      copy_to_lds(src[h] + (size_t)st * 64, to + (uint32_t)h * 4096u, lane_off);
  };
  // operands of v_mfma_f32_32x32x16_f16: lane l supplies 8 consecutive k, the group l / 32 of the
  // 16, of row (or column) l % 32; vectors and centroids use the same split of k over the lanes.
  // The centroids are the rows of the product and the vectors its columns, so that a lane ends up
  // with 16 CA scores of ONE vector per block column and the smallest of them is found in registers.
  struct Operands { halfx8 c[CA], y[2]; };
  auto read = [&](const u32x4 *buf, int kk) {  // 16 of the step's coordinates
    Operands o;
    const int row = lane & 31;  // (block rows start at multiples of 32: same place)
    const int at = row * 4 + ((kk * 2 + (lane >> 5)) ^ place_swap(row & 15));
#pragma unroll
    for (int b = 0; b < 2; ++b) o.y[b] = __builtin_bit_cast(halfx8, buf[(wv * 64 + b * 32) * 4 + at]);
#pragma unroll
    for (int a = 0; a < CA; ++a) o.c[a] = __builtin_bit_cast(halfx8, buf[(kTileM + wc * 32 * CA + a * 32) * 4 + at]);
    __builtin_amdgcn_sched_barrier(0);  // asked for here, in front of the multiplications that follow
    return o;
  };
  auto multiply = [&](const Operands &o) {
#pragma unroll
    for (int a = 0; a < CA; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.c[a], o.y[b], acc[a][b], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Loads come back in order: with as many outstanding as the next step has, this step's are in LDS, the wavefront's
  // own here and everybody's behind the barrier.  Behind it everybody is through with the buffer of the step before as
  // well (its reads have returned: lgkmcnt), which the step after the next takes.
  asm volatile("" :: "v"(bias));  // (the bias has its register before the copies are counted)
  fetch(0);
  if (steps > 1) fetch(1);
  // The multiplications run half a step behind the reads: the second half of a step is multiplied behind the next
  // barrier, while the first half of the next step comes out of LDS.
  Operands first, second;
  for (int st = 0; st < steps; ++st) {
    if (st + 1 < steps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kUnitsY + kUnitsC) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (st + 2 < steps) fetch(st + 2);
    const u32x4 *buf = s_op + (st % kBuffers) * kBuf;
    first = read(buf, 0);
    if (st > 0) multiply(second);
    second = read(buf, 1);
    multiply(first);
  }
  multiply(second);
  if (tid < kTileN) s_cn[tid] = bias;
  __syncthreads();

  // result layout of a 32 x 32 block: register r of lane l holds row (r / 4) * 8 + (l / 32) * 4 + r % 4 (a
  // centroid), column l % 32 (a vector); acc[a][b] is the block of centroid block a and vector block b
  auto centroid_of = [&](int a, int r) { return col0 + wc * 32 * CA + a * 32 + (r / 4) * 8 + (lane >> 5) * 4 + (r % 4); };
  RowMeta mt[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int64_t i = row0 + wv * 64 + b * 32 + (lane & 31);
    mt[b] = meta[i < n ? i : n - 1];
  }
  // scores in place; centroids past the last one score +inf or a NaN (their bias is infinite, their halves are whatever
  // the memory holds), all others less than infinity unless the vector holds a NaN
#pragma unroll
  for (int a = 0; a < CA; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float cn = s_cn[wc * 32 * CA + a * 32 + (r / 4) * 8 + (lane >> 5) * 4 + (r % 4)];
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b][r] = fmaf(-mt[b].scale, acc[a][b][r], cn);
    }
  if (MATRIX) {
    const bool quads = D.nlist % 4 == 0;  // a lane's 4 consecutive centroids of one vector go out as one 16-byte store
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int64_t i = row0 + wv * 64 + b * 32 + (lane & 31);
      if (i >= n) continue;
      float *out = approx + (size_t)i * D.nlist;
#pragma unroll
      for (int a = 0; a < CA; ++a)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
          const int c = centroid_of(a, r);
          if (quads && c + 3 < D.nlist) {
            *reinterpret_cast<float4 *>(out + c) = make_float4(acc[a][b][r], acc[a][b][r + 1], acc[a][b][r + 2], acc[a][b][r + 3]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (c + j < D.nlist) out[c + j] = acc[a][b][r + j];
          }
        }
    }
    return;
  }
  // The tile is reduced here: per vector its smallest score and the centroids within the band of it.
  if (tid < kTileM) s_cnt[tid] = 0u;
  float mine[2];  // smallest score of this lane's vector over the lane's centroids
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    float v = __builtin_inff();
#pragma unroll
    for (int a = 0; a < CA; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) v = fminf(v, acc[a][b][r]);
    mine[b] = v;
    v = fminf(v, __shfl_xor(v, 32));  // the other half of the lanes holds the other centroids of the same vector
    if (lane < 32) s_min[wv * 64 + b * 32 + lane][wc] = v;
  }
  __syncthreads();
  // A lane counts its hits and notes the last one, without a branch; it takes their places with one addition.  Nearly
  // always the hit is its smallest score alone, which is at hand; lanes with several go through the blocks of 32
  // centroids again that hold some.  (A branch and an addition in LDS for every one of the scores, each waited for,
  // were 8 us of the 30 that a tile of 768 dimensions took.)
  uint32_t hits[2][CA], all[2], last[2], slot[2];
  float low[2], limit[2], per[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int row = wv * 64 + b * 32 + (lane & 31);
    // the smallest of the tile plus the band of the vector, a little wider than the refinement's, so that
    // what the refinement asks for is certainly among what is kept here; infinite scores stay out
    low[b] = fminf(s_min[row][0], s_min[row][1]);
    const float width = mt[b].band * 1.01f;
    limit[b] = fminf(low[b] + width, 3.402823466e38f);
    per[b] = width < __builtin_inff() ? 255.f / width : 0.f;
    all[b] = last[b] = 0u;
#pragma unroll
    for (int a = 0; a < CA; ++a) {
      hits[b][a] = 0u;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool hit = acc[a][b][r] <= limit[b];
        hits[b][a] += hit ? 1u : 0u;
        last[b] = hit ? (uint32_t)(a * 16 + r) : last[b];
      }
      all[b] += hits[b][a];
    }
    slot[b] = all[b] ? atomicAdd(&s_cnt[row], all[b]) : (uint32_t)kTileCands;
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int row = wv * 64 + b * 32 + (lane & 31);
    auto keep = [&](float score, uint32_t at, uint32_t to) {
      // how far above the smallest score, in steps of a 255th of the width and rounded down, over the column
      const uint32_t above = (uint32_t)fminf((score - low[b]) * per[b], 255.f);
      const uint32_t col = (uint32_t)(wc * 32 * CA) + (at >> 4) * 32u + ((at & 15u) >> 2) * 8u + (uint32_t)(lane >> 5) * 4u + (at & 3u);
      s_kept[row][to] = (uint16_t)(above << 8 | col);
    };
    if (all[b] == 1u && slot[b] < (uint32_t)kTileCands) keep(mine[b], last[b], slot[b]);
    if (__any(all[b] > 1u)) {  // uniform
      uint32_t to = all[b] > 1u ? slot[b] : (uint32_t)kTileCands;
#pragma unroll
      for (int a = 0; a < CA; ++a)
        if (__any(hits[b][a] && to < (uint32_t)kTileCands))  // uniform
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (acc[a][b][r] <= limit[b] && to < (uint32_t)kTileCands) keep(acc[a][b][r], (uint32_t)(a * 16 + r), to++);
    }
  }
  __syncthreads();
  if (tid < kTileM && row0 + tid < n) {
    const size_t at = (size_t)(row0 + tid) * tc.tiles + col_tile;
    const uint32_t cnt = s_cnt[tid];
    const uint2 *kept = reinterpret_cast<const uint2 *>(s_kept[tid]);
    uint2 *out = reinterpret_cast<uint2 *>(tc.kept + at * kTileCands);
    tc.tmin[at] = fminf(s_min[tid][0], s_min[tid][1]);
    tc.cnt[at] = cnt;
    out[0] = kept[0];
    if (cnt > 4u) out[1] = kept[1];  // (few tiles have so many, and nobody reads what is not counted)
  }
}

// ---- refinement of the assignment.  The smallest approximate score of a row is the
// smallest of its tiles' minima; the centroids within the error band of it (from
// the tiles' kept columns; from all columns of a tile that had more in the band
// than it could keep) are the candidates.  One candidate alone IS the nearest
// centroid, and that is what most rows have.  Where there are more, they are scored
// in the fixed double arithmetic and the best is taken, ties to the lowest index;
// then the next position of the list ("did = atomicAdd(nl_k, 1)").
// A score is a chain of d dependent double operations, and a wavefront issues every
// one of them for all its lanes however few have a candidate: with a wavefront to a
// row and a lane or two at work this was bound by the issue of those instructions
// (21,845 rows of 768 dimensions: 280 us).  So a workgroup reads the digests of up to
// 64 rows first, a few lanes to a row, puts the candidates of the rows that have
// several into a list, and then scores the list: four threads to a candidate while the list is no longer than the
// workgroup, a thread to each where it is.

// exact_score() below with four neighbouring lanes to a candidate (all four call with the same arguments, and all have the
// score): lane s of the four brings chunks s, s + 4, ... and goes on with the chain at each of them, and the sum goes from
// lane to lane with the chain.  (The others' operations at that time are of no use, but a wavefront issues them anyway, and
// the sum moves once per chunk where the terms would move once each: a workgroup's 38 candidates wait for the issue of 2.3
// instructions to a dimension instead of 3.8, or 5 with the conversions of inner products.)  A lane alone waits for a trip
// to memory per eight chunks, 24 of them at 768 dimensions and next to nobody else on the compute unit; here two sets of
// 16 chunks take turns.  (28,928 rows of 768 dimensions, 38 candidates to a workgroup: the refinement 57 us with a lane to
// a candidate and 1,034 workgroups, 45 with four and 998, 35 since the sum moves; in a bulk load of three sub-rounds 31 on
// average.)
template <int S>
__device__ __forceinline__ double quad_take(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, S * 0x55, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), S * 0x55, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double exact_score_quad(const Dev &D, const float *__restrict__ y, int c) {
  const float4 *row4 = reinterpret_cast<const float4 *>(D.centroids + (size_t)c * D.d);
  const float4 *y4 = reinterpret_cast<const float4 *>(y);
  const bool l2 = D.metric == 0;
  const int sub = threadIdx.x & 3, last = D.d4 - 1;
  constexpr int kU = 4;  // chunks of a lane in a set
  double acc = 0.0;
  float4 a0[kU], b0[kU], a1[kU], b1[kU];
  auto load = [&](float4 *a, float4 *b, int j) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int at = min(j + 4 * u + sub, last);
      a[u] = y4[at];
      b[u] = row4[at];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto use = [&](const float4 *a, const float4 *b, int j) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      double p0 = a[u].x, p1 = a[u].y, p2 = a[u].z, p3 = a[u].w, q0 = b[u].x, q1 = b[u].y, q2 = b[u].z, q3 = b[u].w;
      if (l2) {
        p0 = q0 = p0 - q0; p1 = q1 = p1 - q1; p2 = q2 = p2 - q2; p3 = q3 = p3 - q3;
      }
      auto chain = [&](auto tag) {
        constexpr int S = decltype(tag)::value;
        if (j + 4 * u + S > last) return;  // uniform
        double next = __builtin_fma(p0, q0, acc);
        next = __builtin_fma(p1, q1, next);
        next = __builtin_fma(p2, q2, next);
        next = __builtin_fma(p3, q3, next);
        acc = quad_take<S>(next);
      };
      chain(std::integral_constant<int, 0>{}); chain(std::integral_constant<int, 1>{});
      chain(std::integral_constant<int, 2>{}); chain(std::integral_constant<int, 3>{});
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  load(a0, b0, 0);
  for (int j = 0; j <= last; j += 8 * kU) {  // uniform
    load(a1, b1, j + 4 * kU);
    use(a0, b0, j);
    if (j + 4 * kU > last) break;
    load(a0, b0, j + 8 * kU);
    use(a1, b1, j + 4 * kU);
  }
  return acc;
}

__device__ inline double exact_score(const Dev &D, const float *__restrict__ y, int c) {
  // the fixed arithmetic of coarse.hip: one double FMA per dimension, dimensions in order; the
  // 16-byte loads run eight chunks ahead of the chain (a load per turn of the chain, waited for each
  // time, made the chain a sequence of trips to memory)
  const float4 *row4 = reinterpret_cast<const float4 *>(D.centroids + (size_t)c * D.d);
  const float4 *y4 = reinterpret_cast<const float4 *>(y);
  const bool l2 = D.metric == 0;
  double acc = 0.0;
  auto chain = [&](const float4 &a, const float4 &b) {
    if (l2) {
      double t = (double)a.x - (double)b.x; acc = __builtin_fma(t, t, acc);
      t = (double)a.y - (double)b.y; acc = __builtin_fma(t, t, acc);
      t = (double)a.z - (double)b.z; acc = __builtin_fma(t, t, acc);
      t = (double)a.w - (double)b.w; acc = __builtin_fma(t, t, acc);
    } else {
      acc = __builtin_fma((double)a.x, (double)b.x, acc);
      acc = __builtin_fma((double)a.y, (double)b.y, acc);
      acc = __builtin_fma((double)a.z, (double)b.z, acc);
      acc = __builtin_fma((double)a.w, (double)b.w, acc);
    }
  };
  int j = 0;
  for (; j + 8 <= D.d4; j += 8) {
    float4 a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) { a[u] = y4[j + u]; b[u] = row4[j + u]; }
#pragma unroll
    for (int u = 0; u < 8; ++u) chain(a[u], b[u]);
  }
  if (j < D.d4) {  // uniform.  What is left, all of it asked for at once too
    float4 a[8], b[8];
    const int last = D.d4 - 1 - j;
#pragma unroll
    for (int u = 0; u < 7; ++u) { a[u] = y4[j + (u < last ? u : last)]; b[u] = row4[j + (u < last ? u : last)]; }
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (u <= last) chain(a[u], b[u]);  // uniform
  }
  return acc;
}

// What a tile kept of a column (16 bits: steps above the tile's smallest score, column), read again: the column's
// centroid, or -1 if its score is certainly beyond the limit.  The steps were rounded down, and are taken for a hundredth
// shorter here than they were there.
__device__ inline float kept_step(float band) { return band < __builtin_inff() ? band / 255.f : 0.f; }
__device__ inline int kept_column(const TileCands &tc, size_t base, int t, uint32_t j, float low, float step, float limit) {
  const uint32_t k = tc.kept[(base + t) * kTileCands + j];
  return low + (float)(k >> 8) * step <= limit ? t * tc.width + (int)(k & 255u) : -1;
}

constexpr int kRefineThreads = 256;
constexpr int kRefineRows = 64;       // rows of a workgroup at most
// Candidates of a row up to which they go to the workgroup's list, and what the list holds: rows that find it full are
// scored by a wavefront each.  Data in clusters much tighter than the whole, with tens of centroids to a cluster, has
// tens of candidates to a row.  Where a workgroup has few rows the list has room for all columns of a tile that could not
// keep its own, too: a wavefront takes such a tile in four turns, one behind the other.
constexpr int kRefineRowCands = 64, kRefineFewRows = 8, kRefineRowCandsFew = 1024;
constexpr int kRefineList = 2048;

// a score as a key: smaller is better, -0 equal to +0
__device__ inline unsigned long long refine_key(bool l2, double s) {
  const unsigned long long b = (unsigned long long)__double_as_longlong((l2 ? s : -s) + 0.0);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ __launch_bounds__(kRefineThreads) void k_assign_refine(Dev D, int64_t n, const float *__restrict__ Y,
                                                                  const RowMeta *__restrict__ meta, TileCands tc,
                                                                  int rows, int lpr, int reserve,
                                                                  int32_t *__restrict__ assign,
                                                                  uint32_t *__restrict__ did) {
  __shared__ unsigned long long s_key[kRefineRows];  // of the rows whose candidates are listed: their best key ...
  __shared__ int s_col[kRefineRows];                 // ... and the answer of every row
  __shared__ float s_limit[kRefineRows];
  __shared__ int s_hard[kRefineRows];                // rows with more candidates than are listed, or no room in the list
  __shared__ unsigned long long s_lkey[kRefineList];
  __shared__ int s_lcol[kRefineList];
  __shared__ uint8_t s_lrow[kRefineList];
  __shared__ uint32_t s_n, s_hards, s_full;  // s_full: where the first row began that did not fit the list
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t i0 = (int64_t)blockIdx.x * rows;
  const bool l2 = D.metric == 0;
  constexpr int kNone = 0x7fffffff;
  if (tid == 0) { s_n = 0; s_hards = 0; s_full = (uint32_t)kRefineList; }
  if (tid < rows) { s_key[tid] = ~0ull; s_col[tid] = kNone; }
  __syncthreads();
  const int sub = tid & (lpr - 1);
  for (int r0 = 0; r0 < rows; r0 += kRefineThreads / lpr) {  // uniform; the lanes of a row stay together
    const int r = r0 + tid / lpr;
    const int64_t i = i0 + r;
    const bool on = r < rows && i < n;
    const size_t base = (size_t)(on ? i : n - 1) * tc.tiles;
    const float *tmin = tc.tmin + base;
    float m = __builtin_inff();
    for (int t = sub; t < tc.tiles; t += lpr) m = fminf(m, tmin[t]);
    const float band = meta[on ? i : n - 1].band;
    for (int o = lpr / 2; o > 0; o >>= 1) m = fminf(m, __shfl_xor(m, o));
    const float limit = m + band, step = kept_step(band);
    // how many candidates: what a tile near the minimum kept, or all of its columns where it could not keep all its own
    uint32_t mine = 0;
    int first = 0;  // one of the lane's candidates
    for (int t = sub; t < tc.tiles; t += lpr) {
      if (!(tmin[t] <= limit)) continue;
      const uint32_t cnt = tc.cnt[base + t];
      if (cnt > (uint32_t)kTileCands) mine += (uint32_t)min(tc.width, D.nlist - t * tc.width);
      else for (uint32_t j = 0; j < cnt; ++j) {
        const int c = kept_column(tc, base, t, j, tmin[t], step, limit);
        if (c >= 0) { ++mine; first = c; }
      }
    }
    uint32_t upto = mine;  // running sum over the row's lanes
    for (int o = 1; o < lpr; o <<= 1) {
      const uint32_t x = __shfl_up(upto, o);
      if (sub >= o) upto += x;
    }
    const uint32_t total = __shfl(upto, (lane & ~(lpr - 1)) + lpr - 1);
    uint32_t to = 0;
    const bool listed = on && total > 1u && total <= (uint32_t)(rows <= kRefineFewRows ? kRefineRowCandsFew : kRefineRowCands);
    if (listed && sub == 0) to = atomicAdd(&s_n, total);
    to = __shfl(to, lane & ~(lpr - 1));
    if (!on) continue;
    if (total == 1u) {  // nobody to compare it with
      if (mine) s_col[r] = first;
    } else if (total > 1u && (!listed || to + total > (uint32_t)kRefineList)) {
      if (sub == 0) {
        s_limit[r] = limit;
        s_hard[atomicAdd(&s_hards, 1u)] = r;
        if (listed) atomicMin(&s_full, to);  // (whoever reserved behind it did not fit either)
      }
    } else if (mine) {  // to the list
      to += upto - mine;
      for (int t = sub; t < tc.tiles; t += lpr) {
        if (!(tmin[t] <= limit)) continue;
        const uint32_t cnt = tc.cnt[base + t];
        const bool all = cnt > (uint32_t)kTileCands;
        const uint32_t count = all ? (uint32_t)min(tc.width, D.nlist - t * tc.width) : cnt;
        for (uint32_t j = 0; j < count; ++j) {
          const int c = all ? t * tc.width + (int)j : kept_column(tc, base, t, j, tmin[t], step, limit);
          if (c >= 0) {
            s_lcol[to] = c;
            s_lrow[to++] = (uint8_t)r;
          }
        }
      }
    }
  }
  __syncthreads();
  // many candidates, or tiles that could not keep all of theirs: a wavefront to a row
  for (uint32_t h = (uint32_t)wave; h < s_hards; h += kRefineThreads / kWave) {  // uniform over the wavefront
    const int r = s_hard[h];
    const size_t base = (size_t)(i0 + r) * tc.tiles;
    const float limit = s_limit[r], step = kept_step(meta[i0 + r].band);
    const float *y = Y + (i0 + r) * D.d;
    double best_s = l2 ? __builtin_inf() : -__builtin_inf();
    int best_c = kNone;
    auto offer = [&](int c) {
      const double s = exact_score(D, y, c);
      const bool take = s != best_s ? (l2 ? s < best_s : s > best_s) : c < best_c;
      best_s = take ? s : best_s;
      best_c = take ? c : best_c;
    };
    for (int t0 = 0; t0 < tc.tiles; t0 += kWave) {
      const int t = t0 + lane;
      const bool near = t < tc.tiles && tc.tmin[base + t] <= limit;
      const uint32_t cnt = near ? tc.cnt[base + t] : 0u;
      if (near && cnt <= (uint32_t)kTileCands)  // the tile kept all its columns within the band: one lane takes them
        for (uint32_t j = 0; j < cnt; ++j) {
          const int c = kept_column(tc, base, t, j, tc.tmin[base + t], step, limit);
          if (c >= 0) offer(c);
        }
      // a tile with more columns in the band than it could keep: all its columns, shared out over the lanes
      unsigned long long full = __ballot(near && cnt > (uint32_t)kTileCands);
      while (full) {  // uniform
        const int tt = t0 + __ffsll((long long)full) - 1;
        full &= full - 1;
        for (int c = tt * tc.width + lane; c < (tt + 1) * tc.width && c < D.nlist; c += kWave) offer(c);
      }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
      const double s = __shfl_xor(best_s, o);
      const int c = __shfl_xor(best_c, o);
      const bool take = s != best_s ? (l2 ? s < best_s : s > best_s) : c < best_c;
      best_s = take ? s : best_s;
      best_c = take ? c : best_c;
    }
    if (lane == 0) s_col[r] = best_c;
  }
  // the listed candidates (a list longer than the workgroup goes round: the scores of the turns are compared through
  // LDS, keys first, then the lowest index among the equal ones).  Four threads to a candidate while the list is no
  // longer than the workgroup, as it nearly always is; a thread to each where it is, and issue is what bounds it.
  const int entries = (int)min(s_n, s_full);
  auto scored = [&](int e, double s) {
    unsigned long long key = ~0ull;
    if (s == s) {  // a score that does not compare is nobody's best
      key = refine_key(l2, s);
      atomicMin(&s_key[s_lrow[e]], key);
    }
    s_lkey[e] = key;
  };
  if (entries <= kRefineThreads) {  // uniform
    for (int e0 = 0; e0 < entries; e0 += kRefineThreads / 4) {  // uniform
      const int e = e0 + tid / 4;
      if (e0 + wave * (kWave / 4) >= entries) break;  // uniform over the wavefront: the fours stay whole
      const int ee = min(e, entries - 1);
      const double s = exact_score_quad(D, Y + (i0 + s_lrow[ee]) * D.d, s_lcol[ee]);
      if (e < entries && (tid & 3) == 0) scored(e, s);
    }
  } else {
    for (int e = tid; e < entries; e += kRefineThreads) scored(e, exact_score(D, Y + (i0 + s_lrow[e]) * D.d, s_lcol[e]));
  }
  __syncthreads();
  for (int e = tid; e < entries; e += kRefineThreads)
    if (s_lkey[e] != ~0ull && s_lkey[e] == s_key[s_lrow[e]]) atomicMin(&s_col[s_lrow[e]], s_lcol[e]);
  __syncthreads();
  if (tid < rows && i0 + tid < n) {
    int c = s_col[tid];
    if (c == kNone) c = 0;  // no score compared (a vector with a NaN): nothing was better than the first centroid
    assign[i0 + tid] = c;
    if (reserve) did[i0 + tid] = atomicAdd(&D.reserved_len[c], 1u);
  }
}

void launch_centroid_halves(const Dev &D, hipStream_t s) {
  hipLaunchKernelGGL(k_centroid_mean, dim3((unsigned)D.d4), dim3(256), 0, s, D);
  const dim3 grid((unsigned)std::min((D.nlist + kTopWaves - 1) / kTopWaves, 256));
  hipLaunchKernelGGL(k_centroid_top, grid, dim3(kTopThreads), 0, s, D);
  hipLaunchKernelGGL(k_centroid_halves, grid, dim3(kTopThreads), 0, s, D);
}

static void launch_half_rows(const Dev &D, int64_t n, const float *Y, u32x4 *half, RowMeta *meta, hipStream_t s) {
  int lpr = 4;
  while (lpr < kWave && lpr < D.dgroups) lpr *= 2;
  const dim3 grid((unsigned)((n * lpr + 255) / 256)), block(256);
  if (D.dgroups <= lpr) hipLaunchKernelGGL(k_half_rows<1>, grid, block, 0, s, D, n, Y, lpr, half, meta);
  else if (D.dgroups <= 2 * lpr) hipLaunchKernelGGL(k_half_rows<2>, grid, block, 0, s, D, n, Y, lpr, half, meta);
  else hipLaunchKernelGGL(k_half_rows<4>, grid, block, 0, s, D, n, Y, lpr, half, meta);  // d is at most 2048
}

// Wide tiles where they give every compute unit a workgroup, else narrow ones.
static int tile_width(const Dev &D, int64_t n) {
  return (n + kTileM - 1) / kTileM * ((D.nlist + 255) / 256) >= 256 ? 256 : 128;
}
struct TileGrid { unsigned blocks; int die_map; };
static TileGrid tile_grid(const Dev &D, int64_t n, int width) {
  const int64_t cols = (D.nlist + width - 1) / width, rows = (n + kTileM - 1) / kTileM;
  const int64_t padded = (cols + kXcds - 1) / kXcds * kXcds;  // to whole turns of the dies
  if (cols * 8 >= padded * 7) return {(unsigned)(rows * padded), 1};
  return {(unsigned)(rows * cols), 0};
}

static constexpr size_t tile_lds(int ca) { return (size_t)kBuffers * (kTileM + 64 * ca) * kTileK * 2; }

hipError_t allow_large_lds_coarse() {
  hipError_t e = allow_lds(k_coarse_mfma<4, true>, tile_lds(4));
  if (e == hipSuccess) e = allow_lds(k_coarse_mfma<4, false>, tile_lds(4));
  if (e == hipSuccess) e = allow_lds(k_coarse_mfma<2, true>, tile_lds(2));
  if (e == hipSuccess) e = allow_lds(k_coarse_mfma<2, false>, tile_lds(2));
  return e;
}

template <int CA, bool MATRIX>
static void launch_tiles(const Dev &D, const TileGrid &tg, int64_t n, const u32x4 *half, const RowMeta *meta, float *approx,
                         const TileCands &tc, unsigned long long *cursor, uint32_t *zero, int zero_n, hipStream_t s) {
  hipLaunchKernelGGL((k_coarse_mfma<CA, MATRIX>), dim3(tg.blocks), dim3(kMfmaThreads), tile_lds(CA), s, D, n, half, meta, approx, tc,
                     tg.die_map, cursor, zero, zero_n);
}

void launch_coarse_mfma(const Dev &D, int64_t n, const float *Y, u32x4 *half, float *approx,
                        unsigned long long *cursor_to_clear, uint32_t *zero, int zero_n, hipStream_t s) {
  if (n <= 0) return;
  RowMeta *meta = search_row_meta(D, n, half);
  launch_half_rows(D, n, Y, half, meta, s);
  const int width = tile_width(D, n);
  const TileGrid tg = tile_grid(D, n, width);
  const TileCands none{};
  if (width == 256) launch_tiles<4, true>(D, tg, n, half, meta, approx, none, cursor_to_clear, zero, zero_n, s);
  else launch_tiles<2, true>(D, tg, n, half, meta, approx, none, cursor_to_clear, zero, zero_n, s);
}

void launch_coarse_tiles(const Dev &D, int64_t n, const float *Y, u32x4 *half, RowMeta *meta, TileCands &tc,
                         hipStream_t s) {
  if (n <= 0) return;
  launch_half_rows(D, n, Y, half, meta, s);
  // the digests of narrow tiles take twice the room: only as many rows as it holds
  tc.width = n * 2 <= tc.rows ? tile_width(D, n) : 256;
  tc.tiles = (D.nlist + tc.width - 1) / tc.width;
  const TileGrid tg = tile_grid(D, n, tc.width);
  if (tc.width == 256) launch_tiles<4, false>(D, tg, n, half, meta, nullptr, tc, nullptr, nullptr, 0, s);
  else launch_tiles<2, false>(D, tg, n, half, meta, nullptr, tc, nullptr, nullptr, 0, s);
}

void launch_assign_refine(const Dev &D, int64_t n, const float *Y, const RowMeta *meta, const TileCands &tc, bool reserve,
                          int32_t *assign, uint32_t *did, hipStream_t s) {
  if (n <= 0) return;
  // four tiles to a lane, so that a workgroup's rows are a turn or a few of trips to memory; as many rows to a
  // workgroup as leave four workgroups to a compute unit, all there is room for (28 rows of 28,928 to a workgroup were
  // 1,034 of them, and the last ten took the kernel as long again as all others)
  int lpr = 4;
  while (lpr < kWave && lpr * 4 < tc.tiles) lpr *= 2;
  int64_t rows = (n + 1023) / 1024;
  const int64_t turn = kRefineThreads / lpr < kRefineRows ? kRefineThreads / lpr : kRefineRows;  // rows read at a time
  rows = rows < 4 ? 4 : rows > kRefineRows ? kRefineRows : rows;
  if (rows > turn) rows = rows / turn * turn;
  hipLaunchKernelGGL(k_assign_refine, dim3((unsigned)((n + rows - 1) / rows)), dim3(kRefineThreads), 0, s, D, n, Y,
                     meta, tc, (int)rows, lpr, reserve ? 1 : 0, assign, did);
}

}  // namespace rtams
