// What a search request needs between its probe lists and its scan: the pruning bound of every
// query (from a sample of its nearest candidates), the (query, list) pairs grouped by list, and
// the scan's work items, cut and shared out over the XCDs.  One launch, three kinds of workgroup.
#include "bound.h"

namespace rtams {

// ------------------------------------------------------------ pair grouping
// The (query, probed list) pairs of a request are grouped by list, so that the
// scan reads a list once for up to tile_q queries (the scan kernel's choice).  One workgroup:
// prefix sums over the lists of the pair counts, the work-item counts and the
// work, then the item descriptors, the split of the items over the 8 XCDs and
// the grouped pair array.  A work item is (list, segment of seg_groups
// 64-vector groups, tile of up to tile_q of the queries probing the
// list); one wavefront walks it.  The items of one segment follow each other, so
// they run at the same time on the same CU or on its neighbours and the segment
// comes from HBM once.  Segments bound the work of one item, so that long lists
// spread over many wavefronts.  The segment length is the shortest power of two
// for which the request has at most `item_budget` items and no XCD more than
// `max_per_xcd` (the launch of the scan is sized from those two).
constexpr int kSegChoices = 8;  // segment lengths 2, 4, ..., 256 groups (1, 2, ..., 128 where the scan walks groups singly)
constexpr int kLdsEntries = 1024;  // probed lists of a request up to which their entries stay in LDS
constexpr int kListChunk = 16;  // lists a thread of the grouping workgroup handles side by side

// The pairs of the request grouped by list: `grouped` holds, list after list in list order, the
// (query, probe) pairs that probe the list, each at the rank the plan gave it.  One workgroup, beside
// the one that cuts the work items (both derive the same pair starts from the same counters: a
// running sum of the pair counts over the lists, a row of consecutive lists per thread at a time, 16 rows in flight).
// Several workgroups may share the pairs (part `part` of `parts`): each derives all the starts (every
// one of them writes the same numbers to pair_start) and places its own share of the pairs.
__device__ void scatter_pairs(const Dev &D, int nq, int nprobe, int max_nprobe, const SearchScratch &S, int part,
                              int parts) {
  constexpr int kWavesG = kGroupThreads / kWave;
  __shared__ uint32_t s_tot[kListChunk * kWavesG + 1];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint32_t *__restrict__ list_cnt = S.list_cnt;
  uint32_t *__restrict__ pair_start = S.pair_start;
  uint32_t before = 0;  // pairs of the lists in front of the current rows
  for (int lb = 0; lb < D.nlist; lb += kListChunk * kGroupThreads) {  // uniform over the workgroup
    const int rows = min(kListChunk, (D.nlist - lb + kGroupThreads - 1) / kGroupThreads);
    uint32_t c[kListChunk], incl[kListChunk];
#pragma unroll
    for (int t = 0; t < kListChunk; ++t) {
      const int l = lb + t * kGroupThreads + tid;
      c[t] = t < rows && l < D.nlist ? list_cnt[l] : 0u;
    }
#pragma unroll
    for (int t = 0; t < kListChunk; ++t) {
      incl[t] = c[t];
      if (t < rows) {  // uniform
        incl[t] = wave_running_sum(incl[t]);
        if (lane == kWave - 1) s_tot[t * kWavesG + wave] = incl[t];
      }
    }
    __syncthreads();
    if (wave == 0) {  // running sum over the (row, wavefront) totals, in list order
      uint32_t carry = 0;
      const int counts = rows * kWavesG;
      for (int i0 = 0; i0 < counts; i0 += kWave) {
        const uint32_t v = i0 + lane < counts ? s_tot[i0 + lane] : 0u;
        const uint32_t in2 = wave_running_sum(v);
        if (i0 + lane < counts) s_tot[i0 + lane] = carry + in2 - v;
        carry += last_lane(in2);
      }
      if (lane == 0) s_tot[kListChunk * kWavesG] = carry;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kListChunk; ++t)
      if (c[t]) pair_start[lb + t * kGroupThreads + tid] = before + s_tot[t * kWavesG + wave] + incl[t] - c[t];
    before += s_tot[kListChunk * kWavesG];
    __syncthreads();  // the totals are reused by the next rows; the starts are read below by other threads
  }
  // eight independent chains of loads per thread
  const int npairs_all = nq * nprobe;
  const int share = (npairs_all + parts - 1) / parts;
  const int npairs = min(npairs_all, (part + 1) * share);
  for (int base = part * share + tid; base < npairs; base += 8 * kGroupThreads) {
    int l[8];
    uint32_t slot[8], pk[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = base + u * kGroupThreads;
      if (idx < npairs) {
        const int q = idx / nprobe, p = idx - q * nprobe;
        const size_t o = (size_t)q * max_nprobe + p;
        l[u] = S.probe_list[o];
        slot[u] = S.pair_slot[o];
        pk[u] = ((uint32_t)q << 10) | (uint32_t)p;
      } else {
        l[u] = -1;
      }
    }
    uint32_t start[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) start[u] = l[u] >= 0 ? pair_start[l[u]] : 0u;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (l[u] >= 0) S.grouped[start[u] + slot[u]] = pk[u];
  }
}

template <bool HALVES>
__device__ __forceinline__ void group_request(const Dev &D, int nq, int nprobe, int max_nprobe, int k, const float *__restrict__ Q,
                                              uint32_t item_budget, uint32_t max_per_xcd, uint32_t tile_q, uint32_t seg_base,
                                              int min_choice, int scatterers, int sample_parts, const SearchScratch &S) {
  const int tile_shift = 31 - __clz((int)tile_q);  // tiles hold a power of two of queries
  if (blockIdx.x >= 1 && (int)blockIdx.x <= scatterers) {  // uniform over the workgroup: these group the pairs by list
    scatter_pairs(D, nq, nprobe, max_nprobe, S, (int)blockIdx.x - 1, scatterers);
    return;
  }
  // the bound's query and sample keys, or the entries of the probed lists of a small request
  __shared__ __attribute__((aligned(16))) unsigned char s_raw[kBoundLdsBytes];
  static_assert(kBoundLdsBytes >= kLdsEntries * sizeof(uint4), "the entries share the bound's LDS");
  if (blockIdx.x > 0) {  // this one sets the bound of a query
    const uint32_t at = blockIdx.x - 1u - (uint32_t)scatterers, part = at / (uint32_t)nq;
    sample_bound<false, HALVES>(D, (int)(at - part * (uint32_t)nq), nprobe, max_nprobe, k, Q, S, s_raw, part, (uint32_t)sample_parts);
    return;
  }
  __shared__ uint32_t s_a[kGroupThreads / kWave], s_b[kGroupThreads / kWave];  // pairs, items and work of every wavefront's lists
  __shared__ unsigned long long s_c[kGroupThreads / kWave];
  __shared__ uint32_t s_begin[9];
  constexpr uint32_t kHugeItems = 512, kHugeCap = 64;  // lists with this many items: at most so many are spread over the workgroup
  __shared__ uint4 s_huge_pl[kHugeCap];
  __shared__ uint32_t s_huge_ist[kHugeCap];
  __shared__ uint32_t s_nhuge;
  __shared__ uint32_t s_rows[kListChunk * (kGroupThreads / kWave) + 1];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint32_t *__restrict__ list_cnt = S.list_cnt;
  uint4 *__restrict__ tile_desc = S.tile_desc;
  // The entries of the probed lists are written by one thread and read by another several times
  // over: every such hand-over through global memory is a round trip of a microsecond that nothing
  // hides (this workgroup is alone on its CU).  A request that can probe at most kLdsEntries
  // different lists keeps them in LDS.
  const bool lean = (long long)min((long long)D.nlist, (long long)nq * nprobe) <= kLdsEntries;
  uint4 *plist = lean ? reinterpret_cast<uint4 *>(s_raw) : S.plist;
  ScanQueues *Qs = S.queues;
  // the word of an item that says how many pairs it has
  auto pairs_word = [&](uint32_t pairs, uint32_t len, uint32_t sg, uint32_t seg) {
    return HALVES ? half_item_word(pairs, len, sg, seg) : pairs;
  };
  // Cost of a list for the split over the XCDs, per group of 64 vectors: reading it once from HBM
  // (each XCD has its own link to memory) plus the arithmetic of every query that probes it.  On
  // this chip one group's bytes cost about as much as the arithmetic of 12 queries (L2) or 24 (IP).
  const uint32_t byte_weight = D.scan_byte_weight > 0 ? (uint32_t)D.scan_byte_weight : D.metric == 0 ? 12u : 24u;

  // The probed lists, compacted in list order (neighbouring lists sit in neighbouring blocks after a
  // bulk load, and the scan reads faster in that order): entry = {list, first pair, pairs, length}.
  // The pair counters are read a row of consecutive lists (one per thread) at a time, 16 such rows in flight;
  // the place of a probed list among the entries comes from ballots and one small prefix sum.  Lists
  // nobody probes are not looked at again (16,384 lists, 256 x 64 pairs: a quarter of the lists).
  // The visible length of every probed list is read ONCE: an insertion may publish while this kernel
  // runs, and the passes below must agree on the segment counts.  (Each pair's own snapshot was
  // taken earlier, so it is not longer than this one.)
  // Counters and lengths of 16 rows are asked for together, the lengths of all lists: waited for one probed list after
  // the other they were most of this pass (16,384 lists: 27 us).
  uint32_t n_c = 0;
  constexpr int kWavesG = kGroupThreads / kWave;
  for (int lb = 0; lb < D.nlist; lb += kListChunk * kGroupThreads) {  // uniform over the workgroup
    const int rows = min(kListChunk, (D.nlist - lb + kGroupThreads - 1) / kGroupThreads);
    uint32_t c[kListChunk], len[kListChunk];
    unsigned long long flags[kListChunk];
#pragma unroll
    for (int t = 0; t < kListChunk; ++t) {
      c[t] = 0u;
      len[t] = 0u;
      if (t < rows) {  // uniform
        const int l = min(lb + t * kGroupThreads + tid, D.nlist - 1);
        c[t] = list_cnt[l];
        len[t] = __hip_atomic_load(&D.visible_len[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
#pragma unroll
    for (int t = 0; t < kListChunk; ++t) {
      flags[t] = 0ull;
      if (t < rows) {  // uniform
        if (lb + t * kGroupThreads + tid >= D.nlist) c[t] = 0u;
        flags[t] = __ballot(c[t] != 0u);
        if (lane == 0) s_rows[t * kWavesG + wave] = (uint32_t)__popcll(flags[t]);
      }
    }
    __syncthreads();
    if (wave == 0) {  // running sum over the (row, wavefront) counts, in list order
      uint32_t carry = 0;
      const int counts = rows * kWavesG;
      for (int i0 = 0; i0 < counts; i0 += kWave) {
        const uint32_t v = i0 + lane < counts ? s_rows[i0 + lane] : 0u;
        const uint32_t incl = wave_running_sum(v);
        if (i0 + lane < counts) s_rows[i0 + lane] = carry + incl - v;
        carry += last_lane(incl);
      }
      if (lane == 0) s_rows[kListChunk * kWavesG] = carry;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kListChunk; ++t)
      if (c[t])
        plist[n_c + s_rows[t * kWavesG + wave] + (uint32_t)__popcll(flags[t] & ((1ull << lane) - 1ull))] =
            make_uint4((uint32_t)(lb + t * kGroupThreads + tid), 0u, c[t], len[t]);
    n_c += s_rows[kListChunk * kWavesG];
    __syncthreads();  // the counts are reused by the next rows; the entries are read below by other threads
  }
  // From here on a wavefront owns a range of consecutive entries and walks it 64 at a time, lane = entry, so that the
  // loads of a turn are one run of memory (a thread with a few entries of its own side by side touches as many cache
  // lines as it has lanes with every load and store, and this one compute unit is all the chip has at work here:
  // 3,500 probed lists of 4,096, 18,600 items: 37 us in five passes of that kind).  Two passes: the totals of every
  // wavefront's range, then the places of its pairs and items, the cuts and the item descriptors in one go.
  constexpr uint32_t kWaves = kGroupThreads / kWave;
  const uint32_t w0 = (uint32_t)((unsigned long long)n_c * wave / kWaves);
  const uint32_t w1 = (uint32_t)((unsigned long long)n_c * (wave + 1) / kWaves);
  auto entry = [&](uint32_t e) { return e < w1 ? plist[e] : make_uint4(0u, 0u, 0u, 0u); };
  // The shortest segments are tried first and nearly always fit the budget.  Twice the length never makes fewer than half
  // the items, so where they do not, no length in front of the one tried next would have done either.
  int choice = min_choice;
  for (;;) {  // uniform: every thread sees the same totals
    const uint32_t seg = seg_base << choice;
    const int seg_shift = 31 - __clz((int)seg);  // (a power of two)
    auto items_of = [&](const uint4 &pl, uint32_t &groups, uint32_t &tiles) {
      groups = (pl.w + kWave - 1) / kWave;
      tiles = (pl.z + tile_q - 1) >> tile_shift;
      return pl.z ? (groups ? (groups + seg - 1) >> seg_shift : 1u) * tiles : 0u;
    };
    auto work_of = [&](const uint4 &pl, uint32_t groups) {
      return pl.z ? (unsigned long long)(pl.z + byte_weight) * (groups ? groups : 1u) : 0ull;
    };
    uint32_t np = 0, ni = 0;
    unsigned long long wk = 0;
    for (uint32_t eb = w0; eb < w1; eb += 4 * kWave) {  // four turns' loads at a time
      uint4 pl[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) pl[u] = entry(eb + u * kWave + (uint32_t)lane);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t groups, tiles;
        np += pl[u].z;
        ni += items_of(pl[u], groups, tiles);
        wk += work_of(pl[u], groups);
      }
    }
    np = last_lane(wave_running_sum(np));
    ni = last_lane(wave_running_sum(ni));
    wk = last_lane(wave_running_sum(wk));
    if (lane == 0) { s_a[wave] = np; s_b[wave] = ni; s_c[wave] = wk; }
    if (tid < 9) s_begin[tid] = 0u;
    if (tid == 0) s_nhuge = 0;
    __syncthreads();
    uint32_t ps = 0, is = 0, total_items = 0;  // where this wavefront's pairs, items and work start
    unsigned long long ws = 0, total_work = 0;
    for (uint32_t w = 0; w < kWaves; ++w) {
      if ((int)w < wave) { ps += s_a[w]; is += s_b[w]; ws += s_c[w]; }
      total_items += s_b[w];
      total_work += s_c[w];
    }
    if (total_items > item_budget && choice < kSegChoices - 1) {
      int k = 1;
      while (((unsigned long long)item_budget << k) < total_items) ++k;
      choice = min(choice + k, kSegChoices - 1);
      __syncthreads();  // the totals have been read
      continue;
    }
    const bool room = total_items <= S.item_cap;  // (otherwise nothing is written: coarser segments, or no scan at all)
    // Item descriptors.  Most lists have a handful of items: their lane writes them itself.  A list with more is taken
    // by the whole wavefront, the lanes writing its items side by side, and one with very many (a
    // hot list probed by dozens of queries has thousands) by the whole workgroup afterwards.  Inside a list the tiles
    // of one segment follow each other, and the tiles are of (almost) equal size.
    constexpr uint32_t kOwnItems = 16;
    uint4 pl_next = entry(w0 + (uint32_t)lane);
    for (uint32_t eb = w0; eb < w1; eb += kWave) {
      const uint4 got = pl_next;
      pl_next = entry(eb + kWave + (uint32_t)lane);  // the next 64 are on their way while these are written
      uint32_t groups, tiles;
      const uint32_t n = items_of(got, groups, tiles);
      const unsigned long long w = work_of(got, groups);
      const uint32_t psum = wave_running_sum(got.z), isum = wave_running_sum(n);
      const unsigned long long wsum = wave_running_sum(w);
      const uint4 pl = make_uint4(got.x, ps + psum - got.z, got.z, got.w);
      const uint32_t ist = is + isum - n;
      const unsigned long long wst = ws + wsum - w;
      ps += last_lane(psum);
      is += last_lane(isum);
      const unsigned long long wend = ws + last_lane(wsum);
      // XCD x starts at the item at which the work prefix passes x/8 of the total; a cut inside a list: at the item
      // the same share of it ends at
      for (uint32_t x = 1; x < 8; ++x) {
        const unsigned long long cut = total_work * x / 8;
        if (cut < ws || cut >= wend) continue;  // uniform: few turns hold a cut
        if (w && wst <= cut && cut < wst + w) s_begin[x] = ist + (uint32_t)((cut - wst) * n / w);
      }
      ws = wend;
      if (!room) continue;  // uniform
      tiles = tiles ? tiles : 1u;
      const uint32_t small = pl.z / tiles;
      const uint32_t extra = pl.z - small * tiles;  // the first `extra` tiles hold one more
      if (n <= kOwnItems) {
        uint32_t sg = 0, tt = 0;
        for (uint32_t i = 0; i < n; ++i) {
          const uint32_t p_lo = tt * small + min(tt, extra);
          tile_desc[ist + i] = make_uint4(pl.x, pl.y + p_lo, pairs_word(small + (tt < extra ? 1u : 0u), pl.w, sg, seg), sg);
          if (++tt == tiles) { tt = 0; ++sg; }
        }
      }
      // the few lists with very many items are left to the whole workgroup (below)
      bool huge = n >= kHugeItems;
      if (huge) {
        const uint32_t slot = atomicAdd(&s_nhuge, 1u);
        if (slot < kHugeCap) {
          s_huge_pl[slot] = pl;
          s_huge_ist[slot] = ist;
        } else {
          huge = false;  // no room: the wavefront takes it after all
        }
      }
      unsigned long long big = __ballot(n > kOwnItems && !huge);
      while (big) {  // uniform over the wavefront
        const int t = __builtin_ctzll(big);
        big &= big - 1;
        const uint32_t l = (uint32_t)__shfl((int)pl.x, t), pst = (uint32_t)__shfl((int)pl.y, t);
        const uint32_t first = (uint32_t)__shfl((int)ist, t), n_t = (uint32_t)__shfl((int)n, t);
        const uint32_t tiles_t = (uint32_t)__shfl((int)tiles, t);
        const uint32_t small_t = (uint32_t)__shfl((int)small, t), extra_t = (uint32_t)__shfl((int)extra, t);
        const uint32_t len_t = HALVES ? (uint32_t)__shfl((int)pl.w, t) : 0u;
        for (uint32_t i = (uint32_t)lane; i < n_t; i += kWave) {
          const uint32_t sg = i / tiles_t, tt = i - sg * tiles_t;
          const uint32_t p_lo = tt * small_t + min(tt, extra_t);
          tile_desc[first + i] = make_uint4(l, pst + p_lo, pairs_word(small_t + (tt < extra_t ? 1u : 0u), len_t, sg, seg), sg);
        }
      }
    }
    __syncthreads();
    uint32_t begin[9], longest = 0;
    begin[0] = 0u;
#pragma unroll
    for (int x = 1; x < 8; ++x) begin[x] = max(begin[x - 1], s_begin[x]);  // several cuts may fall into one list: keep the sequence monotone
    begin[8] = total_items;
#pragma unroll
    for (int x = 0; x < 8; ++x) longest = max(longest, begin[x + 1] - begin[x]);
    if (longest > max_per_xcd) {  // uniform.  Items of very unequal cost: give every XCD the same number instead
#pragma unroll
      for (int x = 1; x < 8; ++x) begin[x] = (uint32_t)((unsigned long long)total_items * x / 8);
      longest = (total_items + 7) / 8;
    }
    const bool fits = room && longest <= max_per_xcd;
    if (!fits && choice + 1 < kSegChoices + 8) {  // coarser segments (bounded: lengths are 32 bit)
      ++choice;
      __syncthreads();  // the cuts and the totals have been read
      continue;
    }
    if (tid == 0) {
#pragma unroll
      for (int x = 0; x < 9; ++x) Qs->begin[x] = begin[x];
      Qs->seg_groups = fits ? seg : 0u;
      if (!fits) {  // more tiles than the request's item descriptors hold: nothing is scanned, and the caller is told
        atomicCAS(&D.ctrl->search_error, 0, -6);
        D.mirror->search_error = -6;
      }
    }
    if (fits) {
      const uint32_t nh = min(s_nhuge, kHugeCap);
      for (uint32_t h = 0; h < nh; ++h) {  // uniform over the workgroup
        const uint4 pl = s_huge_pl[h];
        const uint32_t first = s_huge_ist[h];
        const uint32_t groups = (pl.w + kWave - 1) / kWave;
        const uint32_t tiles = (pl.z + tile_q - 1) >> tile_shift;
        const uint32_t n = (groups ? (groups + seg - 1) >> seg_shift : 1u) * tiles;
        const uint32_t small = pl.z / tiles, extra = pl.z - small * tiles;
        for (uint32_t i = (uint32_t)tid; i < n; i += kGroupThreads) {
          const uint32_t sg = i / tiles, tt = i - sg * tiles;
          const uint32_t p_lo = tt * small + min(tt, extra);
          tile_desc[first + i] = make_uint4(pl.x, pl.y + p_lo, pairs_word(small + (tt < extra ? 1u : 0u), pl.w, sg, seg), sg);
        }
      }
    }
    break;
  }
}

__global__ __launch_bounds__(kGroupThreads, 4) void k_group(Dev D, int nq, int nprobe, int max_nprobe, int k,
                                                         const float *__restrict__ Q,
                                                         uint32_t item_budget, uint32_t max_per_xcd,
                                                         uint32_t tile_q, uint32_t seg_base, int min_choice, int scatterers, int sample_parts,
                                                         SearchScratch S) {
  group_request<false>(D, nq, nprobe, max_nprobe, k, Q, item_budget, max_per_xcd, tile_q, seg_base, min_choice, scatterers, sample_parts, S);
}
// ... of a request that reads the halves beside the lists: its samples do, too
__global__ __launch_bounds__(kGroupThreads, 4) void k_plan_halves(Dev D, int nq, int nprobe, int max_nprobe, int k,
                                                         const float *__restrict__ Q,
                                                         uint32_t item_budget, uint32_t max_per_xcd,
                                                         uint32_t tile_q, uint32_t seg_base, int min_choice, int scatterers, int sample_parts,
                                                         SearchScratch S) {
  group_request<true>(D, nq, nprobe, max_nprobe, k, Q, item_budget, max_per_xcd, tile_q, seg_base, min_choice, scatterers, sample_parts, S);
}

constexpr int kPqBoundThreads = 1024;

// The bound of every query of a request over quantised lists (the grouping by list that the scan
// of flat lists needs is not made).
// The workgroup of a query first writes the query's table of sub-scores: lut[q][m][c] = squared
// distance (L2) or inner product (IP) between sub-vector m of the query and entry c of codebook m,
// fp32, one FMA chain in the order of the dimensions; the scan reads it from there, its sample from LDS (read back from
// memory, and the nearest list looked up behind it, the launch took 19.1 us for 256 queries, 16 codes to a vector; 14.0 now).
__global__ __launch_bounds__(kPqBoundThreads) void k_pq_bound(Dev D, int nprobe, int max_nprobe, int k,
                                                            const float *__restrict__ Q, SearchScratch S) {
  extern __shared__ float s_lut[];  // [M][256]
  const int q = blockIdx.x;
  const PqNearest nearest = pq_nearest(D, max_nprobe, q, S);
  {
    const int M = D.pq_m, ds = D.d / M;
    const float *__restrict__ yq = Q + (size_t)q * D.d;
    float *__restrict__ lut = S.lut + (size_t)q * M * 256;
    // M * 256 entries, 1024 threads: M / 4 rounds, four of them side by side (their loads overlap);
    // 16-byte loads where the sub-space allows
    for (int i0 = threadIdx.x; i0 < M * 256; i0 += 4 * kPqBoundThreads) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      if (ds % 4 == 0) {  // uniform
        for (int j4 = 0; j4 < ds / 4; ++j4) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = i0 + r * kPqBoundThreads;
            if (i < M * 256) {
              const float4 ev = reinterpret_cast<const float4 *>(D.codebooks + (size_t)i * ds)[j4];
              const float4 yv = reinterpret_cast<const float4 *>(yq + (size_t)(i >> 8) * ds)[j4];
              if (D.metric == 0) {
                const float u0 = ev.x - yv.x, u1 = ev.y - yv.y, u2 = ev.z - yv.z, u3 = ev.w - yv.w;
                acc[r] = fmaf(u0, u0, acc[r]); acc[r] = fmaf(u1, u1, acc[r]);
                acc[r] = fmaf(u2, u2, acc[r]); acc[r] = fmaf(u3, u3, acc[r]);
              } else {
                acc[r] = fmaf(ev.x, yv.x, acc[r]); acc[r] = fmaf(ev.y, yv.y, acc[r]);
                acc[r] = fmaf(ev.z, yv.z, acc[r]); acc[r] = fmaf(ev.w, yv.w, acc[r]);
              }
            }
          }
        }
      } else {
        for (int j = 0; j < ds; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = i0 + r * kPqBoundThreads;
            if (i < M * 256) {
              const float ev = D.codebooks[(size_t)i * ds + j], yv = yq[(size_t)(i >> 8) * ds + j];
              if (D.metric == 0) { const float u = ev - yv; acc[r] = fmaf(u, u, acc[r]); }
              else acc[r] = fmaf(ev, yv, acc[r]);
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (i0 + r * kPqBoundThreads < M * 256) lut[i0 + r * kPqBoundThreads] = s_lut[i0 + r * kPqBoundThreads] = acc[r];
    }
  }
  __syncthreads();  // the sample below reads the table
  __shared__ __attribute__((aligned(16))) unsigned char s_raw[kPqBoundLdsBytes];
  sample_bound<true, false>(D, q, nprobe, max_nprobe, k, nullptr, S, s_raw, 0u, 1u, s_lut, nearest);
}


hipError_t allow_large_lds_group() { return allow_lds(k_pq_bound, 64 * 1024); }

void launch_group(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int k, const float *Q,
                  int item_budget, const SearchScratch &S, hipStream_t s) {
  if (nq <= 0) return;
  if (D.pq_m > 0) {
    // (64 codes to a vector: 64 KiB, and the keys beside them)
    hipLaunchKernelGGL(k_pq_bound, dim3((unsigned)nq), dim3(kPqBoundThreads), (size_t)D.pq_m * 1024, s, D, nprobe, max_nprobe, k, Q, S);
    return;
  }
  // workgroup 0 cuts the work items, the next few group the pairs (one for every 2048 pairs, at most 8:
  // placing a pair is a chain of three round trips to memory), the others set the bound of a query each
  const ScanShape sh = scan_shape(D, item_budget);
  const int64_t pairs = nq * nprobe;
  const int scatterers = (int)(pairs <= 2048 ? 1 : pairs >= 8 * 2048 ? 8 : (pairs + 2047) / 2048);
  // (as many workgroups to a query as are on the chip at once; two are not worth their hand-over)
  const int64_t room = (2 * kComputeUnits - 1 - scatterers) / nq;
  const int parts = room < 3 ? 1 : room > kSampleParts ? kSampleParts : (int)room;
  hipLaunchKernelGGL(D.scan_halves ? k_plan_halves : k_group, dim3(1 + (unsigned)scatterers + (unsigned)(nq * parts)), dim3(kGroupThreads), 0, s, D, (int)nq,
                     nprobe, max_nprobe, k, Q, (uint32_t)item_budget,
                     (uint32_t)(sh.grid / (int)kXcds * sh.items_per_wg), (uint32_t)sh.tile_q, (uint32_t)sh.seg_base, sh.min_choice,
                     scatterers, parts, S);
}

}  // namespace rtams
