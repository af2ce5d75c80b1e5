// What the scans on the matrix cores share: a tile's queries, the staging of survivors on their way out, and how a
// workgroup comes to its work item.
#pragma once
#include "search_common.h"

namespace rtams {

struct TileQuery {  // kMmQueryWords 32-bit words
  uint32_t q, len, bound;
  float qn;
  float unscale;  // narrow lists: what turns a product of the pieces into a product of the query
  uint32_t pad[3];
  uint64_t keys, poss;  // addresses of the query's survivor records (keys, positions)
};
static_assert(sizeof(TileQuery) == kMmQueryWords * 4, "words per query of a tile");

struct HalfTileQuery {  // ... of the scan of halves, which has the rest apart (scan_halves.hip)
  uint64_t keys, poss;
  uint32_t q, pad;
};
static_assert(sizeof(HalfTileQuery) == kHalfQueryWords * 4, "words per query of a tile");

template <int CAP>
struct WaveStageOf {  // survivors of one wavefront on their way out
  uint32_t key[CAP], pos[CAP];
  uint8_t row[CAP];  // which query of the tile
  uint32_t qcnt[kMmTileMax], qbase[kMmTileMax];
};
typedef WaveStageOf<kMmStageCap> WaveStage;
static_assert(sizeof(WaveStage) == kMmStageBytes, "staging bytes per wavefront");
typedef WaveStageOf<kHalfStageCap> HalfStage;
static_assert(sizeof(HalfStage) == kHalfStageBytes, "staging bytes per wavefront");

// The staging area at work: what a wavefront keeps, and its way out.
template <typename Query, int CAP>
struct StagingOf {
  const SearchScratch &S;
  const Query *tq;
  WaveStageOf<CAP> &st;
  uint32_t staged;  // survivors in the area (uniform over the wavefront)
  __device__ __forceinline__ void wave_sync() {  // LDS operations of one wavefront execute in order; keep the compiler from moving them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void flush() {
    const int lane = threadIdx.x & (kWave - 1);
    if (lane < kMmTileMax) st.qcnt[lane] = 0u;
    wave_sync();
    constexpr int kMine = CAP / kWave;
    uint32_t rank[kMine], row[kMine];
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const uint32_t e = (uint32_t)lane + u * kWave;
      row[u] = e < staged ? st.row[e] : 0u;
      rank[u] = e < staged ? atomicAdd(&st.qcnt[row[u]], 1u) : 0u;  // place among the query's survivors of this flush
    }
    wave_sync();
    if (lane < kMmTileMax) {
      const uint32_t c = st.qcnt[lane];
      st.qbase[lane] = c ? atomicAdd(rec_count(S, tq[lane].q), c) : 0u;  // rows past the tile's last query have none
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const uint32_t e = (uint32_t)lane + u * kWave;
      if (e < staged) {
        // (a pointer rebuilt from integers has no address space: say "global", or the stores become FLAT
        // operations, and while one of those is pending every wait of the load pipeline has to be for
        // ALL outstanding memory operations)
        const uint64_t at = 4ull * (st.qbase[row[u]] + rank[u]);
        *(GlobalU32 *)(tq[row[u]].keys + at) = st.key[e];
        *(GlobalU32 *)(tq[row[u]].poss + at) = st.pos[e];
      }
    }
    wave_sync();
    staged = 0;
  }
  // which of the lane's four candidates (bits of `pass`) survive for row `row` of the tile, at places slot, slot + 1, ...
  __device__ __forceinline__ void keep(uint32_t pass, const uint32_t *key, uint32_t slot, uint32_t row) {
    if (__ballot(pass != 0u) == 0ull) return;  // uniform
    // places in the staging area: candidate r of every lane, lane after lane, then candidate r + 1
    uint32_t at[4], total = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned long long m = __ballot((pass >> r) & 1u);
      at[r] = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      total += (uint32_t)__popcll(m);
    }
    if (staged + total > (uint32_t)CAP) flush();  // uniform; at most 4 x 64 at once: they always fit an empty area
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (pass & (1u << r)) {
        const uint32_t e = staged + at[r];
        st.key[e] = key[r];
        st.pos[e] = slot + r;
        st.row[e] = (uint8_t)row;
      }
    staged += total;
  }
  // the lane's vector, at place `slot`, for query `row` of the tile, if `pass`
  __device__ __forceinline__ void keep_one(bool pass, uint32_t key, uint32_t slot, uint32_t row) {
    const unsigned long long m = __ballot(pass);
    if (m == 0ull) return;  // uniform
    const uint32_t total = (uint32_t)__popcll(m);
    if (staged + total > (uint32_t)CAP) flush();  // uniform; at most 64 at once: they always fit an empty area
    if (pass) {
      const uint32_t e = staged + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      st.key[e] = key;
      st.pos[e] = slot;
      st.row[e] = (uint8_t)row;
    }
    staged += total;
  }
};
typedef StagingOf<TileQuery, kMmStageCap> Staging;

// Hardware hands consecutive workgroup ids to the 8 XCDs in turn, so workgroup i runs on XCD i % 8 and
// takes item i / 8 of that XCD's range of items (a contiguous range of lists); workgroups past the end
// of their range leave at once.
// STEAL (long scans): the ranges are cut for equal cost, but the XCDs do not finish together (measured
// at 20 M x 256: the last one 5 to 14 % behind the average), so a workgroup whose XCD has no item left
// for it takes one from the BACK of another XCD's range.  All such workgroups of an XCD go to the same
// victim first (the next XCD that is not done) and get neighbouring items: the tiles of one segment,
// which then come from memory once for this XCD too.  Whoever takes an item, owner or not, takes it
// by swapping the descriptor's pair count for zero, so every item is scanned exactly once; an owner
// that finds its item gone goes looking as well.  A victim whose back has met its front (a swap that
// found zero, or no item left) is marked done and not asked again.  Nobody waits for anybody: a
// workgroup that finds nothing leaves.  Short scans keep the plain mapping: the swap is a round trip
// in front of every item, and the launch has tens of thousands of workgroups that find their range
// used up and should leave at once (measured at 1 M x 128, 2,048 items: 226 instead of 103 us).
// The number of pairs of the workgroup's item, whose descriptor and segment length are left in desc and seg; 0: none.
template <bool STEAL>
__device__ __forceinline__ uint32_t take_item(const SearchScratch &S, uint4 &desc, uint32_t &seg) {
  ScanQueues *Qs = S.queues;
  const uint32_t xcd = blockIdx.x % kXcds;
  const uint32_t own = Qs->begin[xcd] + blockIdx.x / kXcds;
  const bool has_own = own < Qs->begin[xcd + 1];
  if (!STEAL && !has_own) return 0u;
  seg = Qs->seg_groups;
  if (seg == 0) return 0u;
  desc = has_own ? S.tile_desc[own] : make_uint4(0u, 0u, 0u, 0u);  // (STEAL: on its way while thread 0 takes the item)
  uint32_t pairs = desc.z;
  if (STEAL) {
    __shared__ uint32_t s_item, s_pairs;
    if (threadIdx.x == 0) {
      uint32_t item = own, got = 0u;
      if (has_own) got = atomicExch(&S.tile_desc[own].z, 0u);
      if (!got) {
        const uint32_t all = (1u << kXcds) - 1u;
        uint32_t done = __hip_atomic_load(&Qs->done_mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) | (1u << xcd);
        for (uint32_t k = 1; k < kXcds && !got && done != all; ++k) {
          const uint32_t y = (xcd + k) % kXcds;
          if ((done >> y) & 1u) continue;
          const uint32_t count = Qs->begin[y + 1] - Qs->begin[y];
          const uint32_t b = atomicAdd(&Qs->back[y], 1u);
          if (b < count) {
            item = Qs->begin[y + 1] - 1u - b;
            got = atomicExch(&S.tile_desc[item].z, 0u);
          }
          if (!got) {
            atomicOr(&Qs->done_mask, 1u << y);
            done |= 1u << y;
          }
        }
      }
      s_item = item;
      s_pairs = got;
    }
    __syncthreads();
    pairs = s_pairs;
    if (pairs == 0) return 0u;  // uniform over the workgroup
    // (a workgroup without an item of its own computed an `own` beyond its range, which may be the very
    // number of the item it took from the next XCD: what it loaded above was nothing)
    if (!has_own || s_item != own) desc = S.tile_desc[s_item];
  }
  return pairs;
}

}  // namespace rtams
