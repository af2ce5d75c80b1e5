// One workgroup's part of the exact coarse scores: the fixed arithmetic that decides list membership and probe choice.
#pragma once
#include <type_traits>
#include "rtams_launch.h"

namespace rtams {

constexpr int kCoarseThreads = 256;

// is score a better than b, ties to the lower index
__device__ inline bool better_pair(int metric, double a, int ia, double b, int ib) {
  if (a != b) return metric == 0 ? (a < b) : (a > b);
  return ia < ib;
}

// One workgroup: VT vectors (converted to double in LDS) against a range of
// centroids, NC centroids per thread at a time (c and c + 256).  ARGMIN selects
// the epilogue: the best centroid of the range per vector, or all scores.  SHARED: a workgroup of this kernel reads the
// scores of the others.  T threads.
template <int METRIC, int VT, int NC, bool ARGMIN, bool SHARED, int T>
__device__ __forceinline__ void coarse_tile(
    const Dev &D, int64_t n, const float *__restrict__ Y, int splits, double *__restrict__ scores,
    double *__restrict__ pscore, int32_t *__restrict__ pidx, unsigned long long *cursor_to_clear,
    uint32_t *__restrict__ zero, int zero_n) {
  extern __shared__ double ylds[];  // [VT][d]
  const int d = D.d, d4 = D.d4;
  const int64_t v0 = (int64_t)blockIdx.x * VT;
  const int split = blockIdx.y;
  // per-request counters of the search plan start from zero (no memset node on the stream)
  if (cursor_to_clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *cursor_to_clear = 0ull;
  if (zero) {
    const int nthreads = gridDim.x * gridDim.y * T;
    for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * T + threadIdx.x; i < zero_n; i += nthreads)
      zero[i] = 0u;
  }

  for (int t = threadIdx.x; t < VT * d; t += T) {
    int v = t / d, j = t - v * d;
    int64_t row = v0 + v;
    ylds[t] = row < n ? (double)Y[row * d + j] : 0.0;
  }
  __syncthreads();

  // centroid range of this split, in units of one row per thread
  constexpr int kStep = NC * T;  // centroids the workgroup takes at a time
  const int per = ((D.nlist + splits - 1) / splits + kStep - 1) / kStep * kStep;
  const int c_begin = split * per;
  const int c_end = min(D.nlist, c_begin + per);

  // running best per vector; the sentinel loses against every real score
  const double worst = METRIC == 0 ? __builtin_inf() : -__builtin_inf();
  double best_s[VT];
  int best_i[VT];
#pragma unroll
  for (int v = 0; v < VT; ++v) { best_s[v] = worst; best_i[v] = 0x7fffffff; }

  // The centroids stream in from their transposed copy: chunk j of 64 consecutive centroids is 1 KiB,
  // one 16-byte load per lane.  A thread's chain of multiply-adds is sequential in the coordinates, so
  // what hides the trips to memory is how far ahead of the chain the loads run: four sets of kSet
  // chunks go round, three of them in flight while the fourth is used up (a single query against
  // thousands of centroids is nothing but such chains, a few per CU).
  constexpr int kSet = VT <= 2 && NC == 1 ? 8 : 4;
  const float4 *CT = reinterpret_cast<const float4 *>(D.centroids_t);
  const size_t cstride = (size_t)D.nlist;
  for (int c = c_begin + threadIdx.x; c < c_end; c += kStep) {
    double acc[NC][VT];
#pragma unroll
    for (int e = 0; e < NC; ++e)
#pragma unroll
      for (int v = 0; v < VT; ++v) acc[e][v] = 0.0;
    // (a second centroid past the range reads the last centroid: its scores are dropped below)
    const float4 *col[NC];
#pragma unroll
    for (int e = 0; e < NC; ++e) col[e] = CT + min(c + e * T, D.nlist - 1);
    auto load_set = [&](float4 (*set)[kSet], int j0) {
#pragma unroll
      for (int e = 0; e < NC; ++e)
#pragma unroll
        for (int u = 0; u < kSet; ++u) set[e][u] = col[e][(size_t)(j0 + u) * cstride];
      __builtin_amdgcn_sched_barrier(0);  // the loads go out here, not where they are used
    };
    // the vectors' coordinates of chunk j, out of LDS
    auto read_y = [&](double (*y)[4], int j) {
#pragma unroll
      for (int v = 0; v < VT; ++v) {
        const double *p = ylds + v * d + 4 * j;
        y[v][0] = p[0]; y[v][1] = p[1]; y[v][2] = p[2]; y[v][3] = p[3];
      }
    };
    auto fma_chunk = [&](int e, const float4 &cv, const double (*y)[4]) {
      const double c0 = (double)cv.x, c1 = (double)cv.y, c2 = (double)cv.z, c3 = (double)cv.w;
#pragma unroll
      for (int v = 0; v < VT; ++v) {
        if (METRIC == 0) {
          double t0 = y[v][0] - c0; acc[e][v] = __builtin_fma(t0, t0, acc[e][v]);
          double t1 = y[v][1] - c1; acc[e][v] = __builtin_fma(t1, t1, acc[e][v]);
          double t2 = y[v][2] - c2; acc[e][v] = __builtin_fma(t2, t2, acc[e][v]);
          double t3 = y[v][3] - c3; acc[e][v] = __builtin_fma(t3, t3, acc[e][v]);
        } else {
          acc[e][v] = __builtin_fma(y[v][0], c0, acc[e][v]);
          acc[e][v] = __builtin_fma(y[v][1], c1, acc[e][v]);
          acc[e][v] = __builtin_fma(y[v][2], c2, acc[e][v]);
          acc[e][v] = __builtin_fma(y[v][3], c3, acc[e][v]);
        }
      }
    };
    // With one or two vectors to a thread a chunk is four or eight dependent multiply-adds, and a trip
    // to LDS in front of each chunk would take longer than they do: the coordinates of the next
    // chunk are asked for before this one is worked on.
    constexpr bool kAhead = VT <= 2;
    auto use_set = [&](const float4 (*set)[kSet], int j0) {
      if (kAhead) {
        double ya[VT][4], yb[VT][4];
        read_y(ya, j0);
#pragma unroll
        for (int u = 0; u < kSet; u += 2) {
          read_y(yb, j0 + u + 1);
#pragma unroll
          for (int e = 0; e < NC; ++e) fma_chunk(e, set[e][u], ya);
          if (u + 2 < kSet) read_y(ya, j0 + u + 2);
#pragma unroll
          for (int e = 0; e < NC; ++e) fma_chunk(e, set[e][u + 1], yb);
        }
      } else {
#pragma unroll
        for (int u = 0; u < kSet; ++u) {
          double y[VT][4];
          read_y(y, j0 + u);  // once for the thread's centroids
#pragma unroll
          for (int e = 0; e < NC; ++e) fma_chunk(e, set[e][u], y);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int kRing = 4 * kSet;
    const int d4_main = d4 / kRing * kRing;  // chunks that go through the four sets; the rest one at a time
    if (d4_main) {  // uniform
      float4 s0[NC][kSet], s1[NC][kSet], s2[NC][kSet], s3[NC][kSet];
      load_set(s0, 0);
      load_set(s1, kSet);
      load_set(s2, 2 * kSet);
      int j = 0;
#pragma unroll 1
      for (; j + kRing < d4_main; j += kRing) {
        load_set(s3, j + 3 * kSet);
        use_set(s0, j);
        load_set(s0, j + kRing);
        use_set(s1, j + kSet);
        load_set(s1, j + kRing + kSet);
        use_set(s2, j + 2 * kSet);
        load_set(s2, j + kRing + 2 * kSet);
        use_set(s3, j + 3 * kSet);
      }
      load_set(s3, j + 3 * kSet);
      use_set(s0, j);
      use_set(s1, j + kSet);
      use_set(s2, j + 2 * kSet);
      use_set(s3, j + 3 * kSet);
    }
    for (int j = d4_main; j < d4; ++j) {
      double y[VT][4];
      read_y(y, j);
#pragma unroll
      for (int e = 0; e < NC; ++e) fma_chunk(e, col[e][(size_t)j * cstride], y);
    }
#pragma unroll
    for (int e = 0; e < NC; ++e) {
      const int ce = c + e * T;
      if (ce >= c_end) break;
      if (ARGMIN) {
#pragma unroll
        for (int v = 0; v < VT; ++v) {
          const bool take = better_pair(METRIC, acc[e][v], ce, best_s[v], best_i[v]);
          best_s[v] = take ? acc[e][v] : best_s[v];
          best_i[v] = take ? ce : best_i[v];
        }
      } else {
#pragma unroll
        for (int v = 0; v < VT; ++v)
          if (v0 + v < n) {
            double *to = &scores[(size_t)(v0 + v) * D.nlist + ce];
            if (SHARED) __hip_atomic_store(to, acc[e][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *to = acc[e][v];
          }
      }
    }
  }

  if (ARGMIN) {
    // the best of the wavefront's lanes, then of the wavefronts: one barrier for all vectors (a tree over the workgroup
    // with a barrier to each of its steps: 64 vectors x 128 against 1,024 lists 6.1 us for the launch, 5.8 now)
    __shared__ double red_s[VT][T / kWave];
    __shared__ int red_i[VT][T / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int v = 0; v < VT; ++v) {
      auto step = [&](auto tag) {  // (where a step brings nothing, a lane meets itself)
        constexpr int kI = decltype(tag)::value;
        const double sb = wave_step<kI>(best_s[v], best_s[v]);
        const int ib = (int)wave_step<kI>((uint32_t)best_i[v], (uint32_t)best_i[v]);
        const bool take = better_pair(METRIC, sb, ib, best_s[v], best_i[v]);
        best_s[v] = take ? sb : best_s[v];
        best_i[v] = take ? ib : best_i[v];
      };
      step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{}); step(std::integral_constant<int, 2>{});
      step(std::integral_constant<int, 3>{}); step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
      if (lane == kWave - 1) { red_s[v][wave] = best_s[v]; red_i[v][wave] = best_i[v]; }
    }
    __syncthreads();
    const int v = threadIdx.x;  // (a thread of the first wavefront to each vector)
    if (v < VT && v0 + v < n) {
      double s = red_s[v][0];
      int c = red_i[v][0];
#pragma unroll
      for (int w = 1; w < T / kWave; ++w) {
        const bool take = better_pair(METRIC, red_s[v][w], red_i[v][w], s, c);
        s = take ? red_s[v][w] : s;
        c = take ? red_i[v][w] : c;
      }
      pscore[(size_t)(v0 + v) * splits + split] = s;
      pidx[(size_t)(v0 + v) * splits + split] = c == 0x7fffffff ? -1 : c;
    }
  }
}

}  // namespace rtams
