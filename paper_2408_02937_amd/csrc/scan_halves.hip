// The list scan of float lists by the halves beside them, on the 16-bit matrix instructions.
#include "scan_tile.h"

namespace rtams {

// A long scan is bound by the bytes of the lists, and most of what it reads only says that a vector is not among the k
// best.  Halves say that as well: the scan reads those, keeps what could come under its query's bound for all that halves
// leave out (HalfQuery, halves.h), and the selection scores what may be among the k best again from the floats.
// v_mfma_f32_16x16x32_f16: the queries of the tile are the rows of the product and the vectors its columns; lane l supplies
// eight coordinates of query and of vector l % 16, a 16-byte chunk of each, and holds, for vector l % 16 of a block of 16, its
// scores against queries 4 (l / 16) .. + 3; |x'|^2 adds up on the vector unit beside it, a chunk's share to a lane.
// A workgroup takes one item, a tile of up to 32 queries.  Its four wavefronts take units of 32 vectors in turn, four chunks of them
// (2 KiB) to a step.  The steps come straight to LDS, into a ring of the wavefront's own, one at work and the others on
// their way, across the ends of the units: what is in flight takes no registers, and is waited for by count.  (In registers,
// the sets would have to go round in unrolled code, or be moved, which waits for them.)  So nothing else may be loaded into
// vector registers in the loop, or its wait would be for everything in flight: the blocks of the next units are looked up by
// scalar loads.
// What bounds it: HBM.  The scans of floats / of halves, one request at a time: 128 queries against 10 M x 96 544 / 279 us (6.0
// TB/s, what a plain read reaches), 64 against 5 M x 768 627 / 296, 256 against skewed lists of 20 M x 256 2,595 / 1,370 (5.0
// TB/s; 1.034 times its bytes cross HBM), and where the lists fit the last-level cache 256 against 1 M x 128 104 / 55.  Two steps of
// 2 KiB ahead: three, four or steps of 4 KiB leave fewer workgroups on a compute unit, 1.5 to 2 times as long with four.
typedef _Float16 HalfX8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ MfmaAcc half_product(const u32x4 &a, const u32x4 &b, const MfmaAcc &acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(HalfX8, a), __builtin_bit_cast(HalfX8, b), acc, 0, 0, 0);
}

// Entry i of a list's block table by scalar loads (i the same for the whole wavefront).  Only for entries below the length that the plan
// saw: those were out before the plan ended, so no cache of this kernel has them as they were before.  An entry that an insertion
// makes while the scan runs may read as whatever was in its place.
typedef const __attribute__((address_space(4))) int32_t *ScalarInts;
__device__ __forceinline__ int32_t table_dir_scalar(const Dev &D, int list, uint32_t i) {
  return ((ScalarInts)(uintptr_t)D.seg_dir)[(size_t)list * kTableSegs + table_seg(i)];
}
__device__ __forceinline__ uint32_t table_entry_scalar(const Dev &D, int32_t dir, uint32_t i) {
  return (uint32_t)((ScalarInts)(uintptr_t)D.slab)[(size_t)((uint32_t)dir + (i - table_seg_first(table_seg(i))))];
}

// A wavefront's copies: step `quad` of unit u goes out next, into slot `slot` of the ring.
struct HalfCopies {
  const char *x;     // the unit's group
  uint32_t u, quad, slot, in_group;  // ... and the unit's first vector in it
  uint32_t next;     // block of the wavefront's next unit
};
struct HalfItem {
  int list;
  uint32_t u_end;     // units of the list up to which the wavefront goes: the plan's
  uint32_t quads, upb, ring_at;  // steps of a unit; units of a block; LDS address of the wavefront's ring
  uint32_t off, off_last;  // where a lane's chunk lies among those of its 16 vectors, in a step and in the last one of a vector
  uint32_t *places;   // LDS: where the wavefront's n-th unit lies in the pool, at n % kHalfPlaces
};

// the copies go on with unit c.u, in block b
__device__ __forceinline__ void place_unit(const Dev &D, const HalfItem &it, HalfCopies &c, uint32_t b) {
  const uint32_t in = c.u % it.upb;
  c.x = block_halves(D, b) + (size_t)(in / 2u) * ((size_t)D.hchunks * (kWave * 16u));
  c.in_group = in % 2u * kHalfUnit;
  if ((threadIdx.x & (kWave - 1)) == 0) it.places[c.u / kMmWaves % kHalfPlaces] = slot_of(D, b, in * kHalfUnit);
}

// the next step on its way, if there is one: two copies, of 16 vectors each, lane l bringing chunk l / 16 of vector l % 16 (of fewer
// than four chunks the last one again)
__device__ __forceinline__ void copy_step(const Dev &D, const HalfItem &it, HalfCopies &c) {
  if (c.u >= it.u_end) return;  // uniform
  const uint32_t to = it.ring_at + c.slot * kHalfStep, width = min((uint32_t)D.hchunks - 4u * c.quad, 4u);
  const uint32_t off = width == 4u ? it.off : it.off_last;
  const char *x = c.x + (size_t)c.quad * (kWave * 64u) + (size_t)(c.in_group * width) * 16u;
#pragma unroll
  for (uint32_t j = 0; j < 2; ++j) copy_to_lds(x + (size_t)(16u * j * width) * 16u, to + j * (kHalfStep / 2u), off);
  c.slot ^= 1u;
  if (++c.quad < it.quads) return;
  c.quad = 0u;
  c.u += kMmWaves;
  if (c.u >= it.u_end) return;
  place_unit(D, it, c, c.next);
  const uint32_t i = (c.u + kMmWaves) / it.upb;
  if (c.u + kMmWaves < it.u_end) c.next = table_entry_scalar(D, table_dir_scalar(D, it.list, i), i);
}

template <int METRIC, int CB>
__device__ __forceinline__ void scan_units_halves(const Dev &D, const SearchScratch &S, const HalfItem &it, uint32_t u0, HalfCopies &c,
                                                  const char *ring, const char *rows, uint32_t row_bytes, const HalfTileQuery *tq,
                                                  const float *consts, HalfStage &st) {
  const int lane = threadIdx.x & (kWave - 1);
  const int col = lane & 15, kg = lane >> 4;
  const char *my_q = rows + (uint32_t)col * row_bytes + (uint32_t)kg * 16u;
  const char *my_x = ring + lane * 16;
  const float ixs = 1.f / halves_scale(D);
  StagingOf<HalfTileQuery, kHalfStageCap> stage{S, tq, st, 0u};
  if (u0 >= it.u_end) return;  // nothing staged yet
  uint32_t quad = 0, slot = 0;
  MfmaAcc acc[2][CB], sum[2][CB];  // products of at most 64 coordinates, and the sums of those (halves_slack, halves.h)
  float sq[2];
  auto clear = [&]() {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      sq[b] = 0.f;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[b][cb] = sum[b][cb] = (MfmaAcc){0.f, 0.f, 0.f, 0.f};
    }
  };
  clear();
  for (;;) {
    // this step's copies are there: all but those of the steps behind it, or, near the end, all
    static_assert(kHalfRing == 2, "one step of two copies behind this one");
    if (c.u >= it.u_end) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    u32x4 y[CB], a[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) a[b] = *reinterpret_cast<const u32x4 *>(my_x + slot * kHalfStep + 1024 * b);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) y[cb] = *reinterpret_cast<const u32x4 *>(my_q + (uint32_t)(16 * cb) * row_bytes + quad * 64u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read
    slot ^= 1u;
    copy_step(D, it, c);
    if (4u * quad + 4u > (uint32_t)D.hchunks && (int)(4u * quad) + kg >= D.hchunks) {  // chunks past the vector
#pragma unroll
      for (int b = 0; b < 2; ++b) a[b] = (u32x4){0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t two = a[b][w];  // (a bit cast of an element of a vector takes its first)
        sq[b] = __builtin_amdgcn_fdot2(__builtin_bit_cast(Half2, two), __builtin_bit_cast(Half2, two), sq[b], false);
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[b][cb] = half_product(y[cb], a[b], acc[b][cb]);
    }
    ++quad;
    if (quad % 2u == 0u || quad == it.quads) {  // uniform
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[b][cb][r] += acc[b][cb][r];
          acc[b][cb] = (MfmaAcc){0.f, 0.f, 0.f, 0.f};
        }
    }
    if (quad < it.quads) continue;  // uniform
    quad = 0;
    // |x'| or its square of the lane's vector of every block of 16
    float nx[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float n = sq[b] + __shfl_xor(sq[b], 16);
      n += __shfl_xor(n, 32);
      if (METRIC == 0) nx[b] = n < __builtin_inff() ? n * (ixs * ixs) : __builtin_nanf("");  // (a NaN passes below)
      else nx[b] = __builtin_amdgcn_sqrtf(n) * ixs;
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float4 bd = *reinterpret_cast<const float4 *>(consts + 16 * cb + 4 * kg);
      const float4 q0 = *reinterpret_cast<const float4 *>(consts + kMmTileMax + 16 * cb + 4 * kg);
      const float4 q1 = *reinterpret_cast<const float4 *>(consts + 2 * kMmTileMax + 16 * cb + 4 * kg);
      const float bound[4] = {bd.x, bd.y, bd.z, bd.w}, c0[4] = {q0.x, q0.y, q0.z, q0.w}, c1[4] = {q1.x, q1.y, q1.z, q1.w};
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float sc[4];
        bool in[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sc[r] = METRIC == 0 ? fmaf(c1[r], sum[b][cb][r], c0[r] + nx[b]) : fmaf(c1[r], sum[b][cb][r], -c0[r] * nx[b]);
          in[r] = !(sc[r] > bound[r]);
        }
        if (__ballot(in[0] || in[1] || in[2] || in[3]) == 0ull) continue;  // uniform
        const uint32_t v = u0 * kHalfUnit + 16u * b + (uint32_t)col, row = 16u * cb + 4u * (uint32_t)kg;
        const uint32_t place = it.places[u0 / kMmWaves % kHalfPlaces] + (uint32_t)col;
        const uint4 l4 = *reinterpret_cast<const uint4 *>(consts + 3 * kMmTileMax + row);
        const uint32_t len[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool pass = in[r] && v < len[r];  // (rows past the tile's queries have length 0)
          if (pass && !(fabsf(sc[r]) < __builtin_inff())) *rec_flag(S, tq[row + r].q) = 1u;
          stage.keep_one(pass, key_of_float(sc[r] + 0.0f), place + 16u * b, row + r);
        }
      }
    }
    clear();
    u0 += kMmWaves;
    if (u0 >= it.u_end) break;
  }
  if (stage.staged) stage.flush();
}

template <int METRIC, bool STEAL>
__global__ __launch_bounds__(kMmWaves *kWave, 4) void k_scan_halves(Dev D, int max_nprobe, SearchScratch S, int tile_rows) {
  // [wavefronts][kHalfRing] steps, [tile_rows] rows of halves, [tile_rows] HalfTileQuery, bounds and constants, places, [wavefronts] WaveStage
  extern __shared__ float4 lds_halves[];
  uint4 desc;
  uint32_t seg;
  const uint32_t word = take_item<STEAL>(S, desc, seg), pairs = half_item_pairs(word);
  if (pairs == 0) return;  // uniform over the workgroup
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.y);
  const int rows = pairs > 16u ? 32 : 16;
  if (rows > tile_rows) return;  // a descriptor the launch was not sized for: nothing is scanned
  const uint32_t units = half_row_units(D), row_bytes = units * 16u + 16u;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  char *ring_mine = reinterpret_cast<char *>(lds_halves) + (size_t)wave * kHalfRing * kHalfStep;
  char *qs = reinterpret_cast<char *>(lds_halves) + (size_t)kMmWaves * kHalfRing * kHalfStep;
  HalfTileQuery *tq = reinterpret_cast<HalfTileQuery *>(qs + (size_t)tile_rows * row_bytes);
  float *consts = reinterpret_cast<float *>(tq + tile_rows);  // bounds, c0, c1 and lengths, kMmTileMax of each
  uint32_t *places = reinterpret_cast<uint32_t *>(consts + kHalfConsts * kMmTileMax);
  HalfStage &st = reinterpret_cast<HalfStage *>(places + kMmWaves * kHalfPlaces)[wave];
  // the wavefront's first steps are on their way before the tile is set up; up to the length that the plan saw, which is no less
  // than any query of the tile wants, and never past the list's chain, whatever the descriptors say
  HalfItem it;
  it.list = __builtin_amdgcn_readfirstlane((int)desc.x);
  it.quads = (uint32_t)(D.hchunks + 3) / 4u;
  it.upb = (uint32_t)D.groups_per_block * (kWave / kHalfUnit);
  const uint32_t lane = threadIdx.x & (kWave - 1), rest = (uint32_t)D.hchunks - 4u * (it.quads - 1u);
  it.off = lane % 16u * 64u + lane / 16u * 16u;
  it.off_last = (lane % 16u * rest + min(lane / 16u, rest - 1u)) * 16u;
  it.places = places + wave * kHalfPlaces;
  it.ring_at = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_address(ring_mine));
  const uint32_t per_seg = seg * (kWave / kHalfUnit), u_begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.w) * per_seg;
  HalfCopies c{nullptr, u_begin + (uint32_t)wave, 0u, 0u, 0u, 0u};
  // what only the descriptor decides is asked for together: the tile's pairs, the blocks of the list, and where the table has the blocks of the
  // first two units (trips to memory behind one another were 6 us of an item's 18: 1 M x 128, 8 groups to an item)
  constexpr uint32_t kInFlight = 4, kThreads = kMmWaves * kWave;
  const uint32_t total = (uint32_t)rows * units;
  const uint32_t pk = threadIdx.x < pairs ? S.grouped[first + threadIdx.x] : 0u;
  uint32_t row[kInFlight], pk_row[kInFlight];
#pragma unroll
  for (uint32_t u = 0; u < kInFlight; ++u) {
    row[u] = min((threadIdx.x + u * kThreads) / units, (uint32_t)rows);
    pk_row[u] = row[u] < pairs ? S.grouped[first + row[u]] : 0u;
  }
  const uint32_t blocks = D.nblk[it.list], planned = u_begin + (uint32_t)__builtin_amdgcn_readfirstlane((int)half_item_units(word));
  const uint32_t i0 = min(c.u, planned) / it.upb, i1 = min(c.u + kMmWaves, planned) / it.upb;
  const int32_t dir0 = table_dir_scalar(D, it.list, i0), dir1 = table_dir_scalar(D, it.list, i1);
  it.u_end = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(blocks * it.upb, planned));
  if (c.u < it.u_end) {  // uniform over the wavefront
    const uint32_t b0 = table_entry_scalar(D, dir0, i0);
    if (c.u + kMmWaves < it.u_end) c.next = table_entry_scalar(D, dir1, i1);
    place_unit(D, it, c, b0);
    for (uint32_t i = 0; i < kHalfRing; ++i) copy_step(D, it, c);
  }
  // the tile's queries: halves (the workgroup together; rows past the last are zero), and words (one thread per row)
  u32x4 v[kInFlight];
  auto fetch = [&](uint32_t base) {
#pragma unroll
    for (uint32_t u = 0; u < kInFlight; ++u)
      v[u] = row[u] < pairs ? half_query_row(D, S, pk_row[u] >> 10)[base + u * kThreads - row[u] * units] : (u32x4){0u, 0u, 0u, 0u};
  };
  auto put = [&](uint32_t base) {
#pragma unroll
    for (uint32_t u = 0; u < kInFlight; ++u)
      if (row[u] < (uint32_t)rows) *reinterpret_cast<u32x4 *>(qs + row[u] * row_bytes + (base + u * kThreads - row[u] * units) * 16u) = v[u];
  };
  fetch(threadIdx.x);
  if ((int)threadIdx.x < rows) {
    HalfTileQuery t{};
    uint32_t len_q = 0u;
    float bound = -__builtin_inff(), c0 = 0.f, c1 = 0.f;
    if (threadIdx.x < pairs) {
      t.q = pk >> 10;
      len_q = S.probe_len[(size_t)t.q * max_nprobe + (pk & 1023u)];
      const unsigned long long qb = S.qbase[t.q];
      t.keys = (uint64_t)(uintptr_t)rec_keys_of(S, qb);
      t.poss = (uint64_t)(uintptr_t)rec_poss_of(S, qb);
      const HalfQuery m = half_query(D, S, t.q);
      bound = l2_score_of_key(halves_bound_key(D, S.bound[t.q], m));  // ("keep everything" is a NaN, which nothing is greater than)
      c0 = m.a;
      c1 = (METRIC == 0 ? -2.f : -1.f) * m.unscale;
    }
    tq[threadIdx.x] = t;
    consts[threadIdx.x] = bound;
    consts[kMmTileMax + threadIdx.x] = c0;
    consts[2 * kMmTileMax + threadIdx.x] = c1;
    reinterpret_cast<uint32_t *>(consts)[3 * kMmTileMax + threadIdx.x] = len_q;
  }
  put(threadIdx.x);
  for (uint32_t base = threadIdx.x + kInFlight * kThreads; base < total; base += kInFlight * kThreads) {
#pragma unroll
    for (uint32_t u = 0; u < kInFlight; ++u) {
      row[u] = min((base + u * kThreads) / units, (uint32_t)rows);
      pk_row[u] = row[u] < pairs ? S.grouped[first + row[u]] : 0u;
    }
    fetch(base);
    put(base);
  }
  __syncthreads();
  // no barrier from here on: the wavefronts only read the tile
  if (rows == 16) scan_units_halves<METRIC, 1>(D, S, it, u_begin + (uint32_t)wave, c, ring_mine, qs, row_bytes, tq, consts, st);
  else scan_units_halves<METRIC, 2>(D, S, it, u_begin + (uint32_t)wave, c, ring_mine, qs, row_bytes, tq, consts, st);
}

typedef void (*HalvesKernel)(Dev, int, SearchScratch, int);
static const HalvesKernel halves_kernels[2][2] = {{k_scan_halves<0, false>, k_scan_halves<0, true>},
                                                  {k_scan_halves<1, false>, k_scan_halves<1, true>}};

hipError_t allow_large_lds_scan_halves() {  // (wide vectors only)
  hipError_t e = hipSuccess;
  for (int i = 0; i < 4 && e == hipSuccess; ++i) e = allow_lds(halves_kernels[i / 2][i % 2], kMmLdsMax);
  return e;
}

void launch_scan_halves(const Dev &D, const ScanShape &sh, int max_nprobe, const SearchScratch &S, hipStream_t s) {
  hipLaunchKernelGGL(halves_kernels[D.metric][D.scan_steal ? 1 : 0], dim3((unsigned)sh.grid), dim3((unsigned)sh.threads), sh.lds, s, D,
                     max_nprobe, S, sh.tile_q);
}

}  // namespace rtams
