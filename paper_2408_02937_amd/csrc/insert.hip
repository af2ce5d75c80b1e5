// Insertion path (Insertion algorithm of the paper): slot reservation with an
// atomic counter per list, lock-free opening and linking of the blocks that do
// not exist yet, in-place fill in the interleaved layout, and publication of
// the batch together with the Exceed() test.
//
// The paper runs all of this in one thread block and separates "reserve",
// "open" and "fill" with two barriers, which only works while a batch cannot
// need two new blocks for one list.  Here the phases of a large batch are
// stream-ordered kernels, so any batch size and any block size work across the
// whole chip, and a batch of up to kTailVecs vectors whose positions the exact
// coarse kernel leaves open, or which are few enough to move, goes through one workgroup
// with barriers, as the paper has it, however many blocks it needs; the
// rule that the block of position did lives at chain index did / T_m, offset
// did % T_m, and that exactly one party opens each new block, is the paper's.
#include "rtams_launch.h"

namespace rtams {

__device__ inline void raise_error(const Dev &D, int code) {
  atomicCAS(&D.ctrl->error, 0, code);
  D.mirror->error = code;
}

// (read past the caches of the compute unit: another thread of the same workgroup may just have raised it)
__device__ inline bool pool_failed(const Dev &D) {
  return __hip_atomic_load(&D.ctrl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// ---- reserve: finish the arg-min over the centroid splits, then take the next
// position of that list ("did = atomicAdd(nl_k, 1)").
__device__ inline int best_of_splits(const Dev &D, int64_t i, int splits, const double *__restrict__ pscore,
                                     const int32_t *__restrict__ pidx) {
  double bs = 0.0;
  int bi = -1;
  for (int s = 0; s < splits; ++s) {
    int ci = pidx[i * splits + s];
    if (ci < 0) continue;
    double cs = pscore[i * splits + s];
    bool better = bi < 0 || (cs != bs ? (D.metric == 0 ? cs < bs : cs > bs) : ci < bi);
    if (better) { bs = cs; bi = ci; }
  }
  return bi < 0 ? 0 : bi;  // no score compared (a vector with a NaN): nothing was better than the first centroid
}

__global__ __launch_bounds__(256) void k_reserve(Dev D, int64_t n, int splits,
                                                 const double *__restrict__ pscore,
                                                 const int32_t *__restrict__ pidx, int reserve,
                                                 int32_t *__restrict__ assign,
                                                 uint32_t *__restrict__ did) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int bi = best_of_splits(D, i, splits, pscore, pidx);
  assign[i] = bi;
  if (reserve) did[i] = atomicAdd(&D.reserved_len[bi], 1u);
}

// ---- reservation in input order.  The atomic reservation above hands out the positions of a
// batch inside a list in arrival order, which is any order (Algorithm 2 takes `did` from an
// atomicAdd as well).  This variant gives the vectors of a batch that fall into one list
// consecutive positions in the order in which they stand in the batch, which is what inserting
// them one at a time would do: the lists then hold the same SEQUENCE on every run.  One thread per
// list walks the batch's assignments (every lane of a wavefront reads the same word).
__global__ __launch_bounds__(256) void k_reserve_ordered(Dev D, int64_t n, const int32_t *__restrict__ assign,
                                                         uint32_t *__restrict__ did) {
  const int list = blockIdx.x * blockDim.x + threadIdx.x;
  if (list >= D.nlist) return;
  uint32_t at = D.reserved_len[list];
  const uint32_t before = at;
  for (int64_t i = 0; i < n; ++i)
    if (assign[i] == list) did[i] = at++;
  if (at != before) D.reserved_len[list] = at;
}

// ---- open.  Positions visible_len .. reserved_len-1 of a list were reserved by this batch; every block index in
// [nblk, ceil(reserved/T_m)) is opened here: table segments first, then blocks from the free stack or the
// bump pointer ("P[atomicAdd(cur_P, 1)]"), headers linked behind the chain.  A workgroup of T threads opens the
// blocks of up to T different lists, one to a thread (list -1: none): it takes the blocks and table entries of all
// of them with one atomic each (an atomic per list on the same two words took 0.2 ms where a first batch touched
// 16,384 lists), and its threads share out the new blocks, whoever's list they are for.
constexpr int kBatchThreads = 128;
template <int T>
struct OpenShared {
  uint32_t first[T];   // new blocks of the threads before
  int32_t list[T], old_last[T];
  uint32_t nb_old[T];
  uint32_t wave_blocks[T / kWave], wave_slab[T / kWave];
  int32_t f_old;       // free_top before the pop
  uint32_t from_stack, base, slab_base, failed;
};

// nb_old: the list's blocks so far, newlen: its length with this batch.  Returns whether there were blocks to open.
template <int T>
__device__ bool wg_open(const Dev &D, int list, uint32_t nb_old, uint32_t newlen, OpenShared<T> &sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint32_t Tm = (uint32_t)D.T_m;
  uint32_t nb_new = 0, count = 0, slab = 0;
  if (list >= 0) {
    nb_new = (newlen + Tm - 1) / Tm;
    if (nb_new > nb_old) {
      count = nb_new - nb_old;
      for (int g = table_seg(nb_old); g <= table_seg(nb_new - 1); ++g)
        if (D.seg_dir[(size_t)list * kTableSegs + g] < 0) slab += (uint32_t)kTableBase << g;
    }
  }
  uint32_t blocks_to = wave_running_sum(count), slab_to = wave_running_sum(slab);
  if (lane == kWave - 1) { sh.wave_blocks[wave] = blocks_to; sh.wave_slab[wave] = slab_to; }
  __syncthreads();
  uint32_t total = 0, slab_total = 0;
  for (int w = 0; w < T / kWave; ++w) {
    if (w < wave) { blocks_to += sh.wave_blocks[w]; slab_to += sh.wave_slab[w]; }
    total += sh.wave_blocks[w];
    slab_total += sh.wave_slab[w];
  }
  if (total == 0) return false;  // uniform over the workgroup
  if (tid == 0) {
    sh.failed = pool_failed(D) ? 1u : 0u;
    if (!sh.failed) {
      const int f = atomicSub(&D.ctrl->free_top, (int)total);
      const int got = f < 0 ? 0 : (f < (int)total ? f : (int)total);
      if (got < (int)total) atomicAdd(&D.ctrl->free_top, (int)total - got);  // give back what was not there
      sh.f_old = f;
      sh.from_stack = (uint32_t)got;
      const uint32_t rem = total - (uint32_t)got;
      sh.base = rem ? atomicAdd(&D.ctrl->cur_P, rem) : 0u;
      sh.slab_base = slab_total ? atomicAdd(&D.ctrl->slab_cur, slab_total) : 0u;
      // backstop only: the host refuses batches that might not fit
      if ((rem && (uint64_t)sh.base + rem > D.nblocks) || (slab_total && (uint64_t)sh.slab_base + slab_total > D.slab_cap)) {
        sh.failed = 1u;
        raise_error(D, -3);
      }
    }
  }
  __syncthreads();
  if (sh.failed) return true;  // uniform
  sh.first[tid] = blocks_to - count;
  sh.list[tid] = list;
  sh.nb_old[tid] = nb_old;
  sh.old_last[tid] = -1;
  if (count) {
    uint32_t off = sh.slab_base + slab_to - slab;
    for (int g = table_seg(nb_old); g <= table_seg(nb_new - 1); ++g) {
      int32_t *dir = &D.seg_dir[(size_t)list * kTableSegs + g];
      if (*dir < 0) { *dir = (int32_t)off; off += (uint32_t)kTableBase << g; }
    }
    if (nb_old > 0) sh.old_last[tid] = *table_entry(D, list, nb_old - 1);
  }
  __syncthreads();
  auto block_of = [&](uint32_t b) -> int32_t {  // b-th new block of this workgroup
    return b < sh.from_stack ? D.free_stack[sh.f_old - 1 - (int)b] : (int32_t)(sh.base + (b - sh.from_stack));
  };
  for (uint32_t b = (uint32_t)tid; b < total; b += T) {
    int lo = 0, hi = T - 1;  // whose block it is: the last thread whose blocks start at or before b
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sh.first[mid] <= b) lo = mid; else hi = mid - 1;
    }
    const uint32_t jl = b - sh.first[lo], bi = sh.nb_old[lo] + jl;
    const bool more = b + 1 < total && (lo == T - 1 || sh.first[lo + 1] > b + 1);
    const int32_t me = block_of(b), before = jl > 0 ? block_of(b - 1) : sh.old_last[lo];
    BlockHeader *h = block_header(D, (uint32_t)me);
    h->prev = before;
    h->next = more ? block_of(b + 1) : -1;
    h->owner = sh.list[lo];
    h->seq = (int32_t)bi;
    h->capacity = (int32_t)Tm;
    h->size = 0;
    *table_entry(D, sh.list[lo], bi) = me;
    if (jl == 0 && before >= 0) block_header(D, (uint32_t)before)->next = me;
  }
  if (count) D.nblk[list] = nb_new;
  return true;
}

// The longest list with this batch, a list's new length to a thread (0: none).  The lengths are final once the positions
// are reserved, so this is done in front of the publication, whose one reporting thread then tells the host: a word of
// host memory that every wavefront with a longer list wrote for itself could keep the smaller of two, and did not get
// its due until some list grew past the larger.  `known`: ctrl->max_len as of any time before (it only grows).
__device__ inline void note_longest(const Dev &D, uint32_t newlen, uint32_t known) {
  if (!__any(newlen > known)) return;  // uniform over the wavefront
  newlen = wave_reduce_last(newlen, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) atomicMax(&D.ctrl->max_len, newlen);
}

// `start`, where the fill goes by lists: the new vectors of list l are start[l] .. of the batch in the order of the fill,
// list after list (which list comes first is as the workgroups arrive, and does not matter).
__global__ __launch_bounds__(256) void k_open(Dev D, uint32_t *__restrict__ start) {
  __shared__ OpenShared<256> sh;
  const int list = blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = list < D.nlist;
  const uint32_t newlen = on ? D.reserved_len[list] : 0u;
  if (start) {  // uniform
    __shared__ uint32_t s_sum[4], s_base;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t added = on ? newlen - D.visible_len[list] : 0u;
    uint32_t upto = wave_running_sum(added);
    if (lane == kWave - 1) s_sum[wave] = upto;
    __syncthreads();
    if (threadIdx.x == 0) s_base = atomicAdd(&D.ctrl->fill_cur, s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
    __syncthreads();
    for (int w = 0; w < wave; ++w) upto += s_sum[w];
    if (on) start[list] = s_base + upto - added;
  }
  note_longest(D, newlen, D.ctrl->max_len);
  wg_open<256>(D, on ? list : -1, on ? D.nblk[list] : 0u, newlen, sh);
}

// ---- fill: chunk c (16 bytes: 4 floats, 8 halves or 16 bytes) of a vector, as the lists keep it
__device__ __forceinline__ float4 stored_chunk(int storage, const float4 *__restrict__ y, int c) {
  if (storage == 1) {
    const float4 a = y[2 * c], e = y[2 * c + 1];
    return make_float4(__uint_as_float(pack_halves(a.x, a.y)), __uint_as_float(pack_halves(a.z, a.w)),
                       __uint_as_float(pack_halves(e.x, e.y)), __uint_as_float(pack_halves(e.z, e.w)));
  }
  if (storage == 2)
    return make_float4(__uint_as_float(pack_bytes(y[4 * c])), __uint_as_float(pack_bytes(y[4 * c + 1])),
                       __uint_as_float(pack_bytes(y[4 * c + 2])), __uint_as_float(pack_bytes(y[4 * c + 3])));
  return y[c];
}

// thread (vector i, chunk c) writes the chunk to its slot; the thread of chunk 0 also writes the id
// (Number: 32 bits where the chunks can be counted in them; a division of 64-bit numbers is most of such a thread's instructions)
template <typename Number>
__global__ __launch_bounds__(256) void k_fill(Dev D, Number chunks, const float *__restrict__ Y,
                                              const int64_t *__restrict__ ids, int64_t id_base,
                                              const int32_t *__restrict__ assign,
                                              const uint32_t *__restrict__ did) {
  const Number t = (Number)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= chunks) return;
  const Number i = t / (Number)D.vchunks;
  const int c = (int)(t - i * (Number)D.vchunks);
  int list = assign[i];
  uint32_t pos = did[i];
  const float scale = D.halves_stride ? halves_scale(D) : 1.f;
  const uint32_t known = D.halves_stride ? D.ctrl->half_inexact : 1u;
  uint32_t mid = pos / (uint32_t)D.T_m, moff = pos % (uint32_t)D.T_m;
  if (mid >= D.nblk[list]) return;  // the block could not be opened (pool exhausted)
  uint32_t b = (uint32_t)*table_entry(D, list, mid);
  const float4 v = stored_chunk(D.storage, reinterpret_cast<const float4 *>(Y) + (size_t)i * D.d4, c);
  block_vecs(D, b)[vec_chunk_index(D, moff, c)] = v;
  if (D.halves_stride) {  // uniform
    bool exact = true;
    put_halves(D, b, moff, c, v, scale, exact);
    if (!exact && !known) D.ctrl->half_inexact = 1u;
  }
  if (c == 0) block_ids(D, b)[moff] = ids ? ids[i] : id_base + i;
}

// ... or, for large batches, list by list.  A vector's chunks lie 1 KiB apart in its group, so a thread's store above is 16
// bytes of a cache line that belong to it alone, and the vectors of one list, which share those lines, are anywhere in the
// batch: 65,536 x 768 took 228 us for 400 MB.  So the batch is put in the order of its lists first (k_fill_order: source
// and place of every vector; ids go out here), and a workgroup takes 64 consecutive ones, 16 chunks of each: 256 bytes
// of a vector at a time into LDS, and out of it with consecutive places side by side, as many to a cache line as the
// batch has for the list: 65,536 x 768 into 8,192 lists 124 us behind 7 for the order.  A run of a list ends inside a line of memory
// that the next one goes on with, so neighbouring runs go to one XCD, and the vectors, which nobody reads again, are read past the
// caches, where the lines wait for their other halves: with the halves beside the lists, half as much again to write, 154 us
// without the two, 131 with the second and 129 with both.
__global__ __launch_bounds__(256) void k_fill_order(Dev D, int64_t n, const int64_t *__restrict__ ids, int64_t id_base,
                                                    const int32_t *__restrict__ assign, const uint32_t *__restrict__ did,
                                                    const uint32_t *__restrict__ start, uint2 *__restrict__ order) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int list = assign[i];
  const uint32_t pos = did[i], mid = pos / (uint32_t)D.T_m, moff = pos % (uint32_t)D.T_m;
  const uint32_t at = start[list] + (pos - D.visible_len[list]);
  if (at >= (uint32_t)n) return;  // (cannot be: the lists' new vectors are the batch)
  uint2 to = make_uint2(~0u, 0u);
  if (mid < D.nblk[list]) {  // (otherwise the block could not be opened: pool exhausted)
    const uint32_t b = (uint32_t)*table_entry(D, list, mid);
    to = make_uint2((uint32_t)i, slot_of(D, b, moff));
    block_ids(D, b)[moff] = ids ? ids[i] : id_base + i;
  }
  order[at] = to;
}

constexpr int kFillSlots = 64, kFillChunks = 16;
constexpr unsigned kFillXcds = 8;
template <int ST>
__global__ __launch_bounds__(256) void k_fill_lists(Dev D, int64_t n, const float *__restrict__ Y,
                                                    const uint2 *__restrict__ order) {
  __shared__ float4 tile[kFillSlots][kFillChunks + 1];  // (the odd row length spreads a column over the banks)
  __shared__ uint2 s_at[kFillSlots];
  const int tid = threadIdx.x;
  const uint32_t of_xcd = gridDim.x / kFillXcds;
  const int64_t s0 = (int64_t)(blockIdx.x % kFillXcds * of_xcd + blockIdx.x / kFillXcds) * kFillSlots;
  const int c0 = (int)blockIdx.y * kFillChunks, chunks = min(kFillChunks, D.vchunks - c0);
  if (tid < kFillSlots) s_at[tid] = s0 + tid < n ? order[s0 + tid] : make_uint2(~0u, 0u);
  __syncthreads();
  {
    const int c = tid % kFillChunks;
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t i = s_at[tid / kFillChunks + 16 * u].x;
      const bool on = i != ~0u && c < chunks;
      if (ST == 0) {
        typedef float Floats __attribute__((ext_vector_type(4)));
        Floats z = {0.f, 0.f, 0.f, 0.f};
        if (on) z = __builtin_nontemporal_load(reinterpret_cast<const Floats *>(Y) + (size_t)i * D.d4 + c0 + c);
        v[u] = make_float4(z.x, z.y, z.z, z.w);
      } else {
        v[u] = on ? stored_chunk(ST, reinterpret_cast<const float4 *>(Y) + (size_t)i * D.d4, c0 + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) tile[tid / kFillChunks + 16 * u][c] = v[u];
  }
  __syncthreads();
  {
    const int slot = tid & (kFillSlots - 1);
    const uint2 at = s_at[slot];
    if (at.x != ~0u) {
      const uint32_t b = at.y / (uint32_t)D.T_m, moff = at.y - b * (uint32_t)D.T_m;
      float4 *to = block_vecs(D, b) + vec_chunk_index(D, moff, c0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = tid / kFillSlots + 4 * u;
        if (c < chunks) to[(size_t)c * kWave] = tile[slot][c];
      }
    }
  }
  if (ST != 0 || D.halves_stride == 0) return;  // uniform
  // four lanes to a vector: 64 bytes of halves side by side
  const int slot = tid / 4;
  const uint2 at = s_at[slot];
  if (at.x == ~0u) return;
  const uint32_t known = D.ctrl->half_inexact;
  const float scale = halves_scale(D);
  bool exact = true;
  const uint32_t b = at.y / (uint32_t)D.T_m, moff = at.y - b * (uint32_t)D.T_m;
  char *half = block_halves(D, b);
#pragma unroll
  for (int u = 0; u < kFillChunks / 8; ++u) {
    const int h = (tid & 3) + 4 * u;
    if (2 * h >= chunks) break;
    const uint2 lo = pack_four_halves(tile[slot][2 * h], scale, exact);
    const uint2 hi = 2 * h + 1 < chunks ? pack_four_halves(tile[slot][2 * h + 1], scale, exact) : make_uint2(0u, 0u);
    *reinterpret_cast<u32x4 *>(half + half_chunk_at(D, moff, (uint32_t)(c0 / 2 + h))) = u32x4{lo.x, lo.y, hi.x, hi.y};
  }
  if (!exact && !known) D.ctrl->half_inexact = 1u;
}

// ---- publish: makes the batch visible and evaluates Exceed() (the equation defining it: vectors appended since the
// last rearrangement, strictly greater than T_m'), a list to a thread of the workgroup (list -1: none).  Everything
// a list needs is asked for at once; the sums over the lists go out with one atomic per wavefront (one per list on
// the same words, a chain of round trips per list and words written to host memory in front of the fences made
// this the longest of the insertion kernels); and what the host is told is written last.
__device__ inline void wg_publish(const Dev &D, int list) {
  const uint32_t T = (uint32_t)D.T_m;
  uint32_t added = 0, told_exceed = 0;
  if (list >= 0) {
    const uint32_t newlen = D.reserved_len[list], old = D.visible_len[list], on0 = D.online[list];
    const bool exceeds = D.exceed[list] != 0, failed = pool_failed(D);
    if (newlen != old && failed) {  // the batch is dropped as a whole
      D.reserved_len[list] = old;
    } else if (newlen != old) {
      for (uint32_t bi = old / T; bi <= (newlen - 1) / T; ++bi) {
        uint32_t b = (uint32_t)*table_entry(D, list, bi);
        uint32_t sz = newlen - bi * T;
        block_header(D, b)->size = (int32_t)(sz < T ? sz : T);
      }
      added = newlen - old;
      D.online[list] = on0 + added;
      if (D.T_mp > 0 && (int64_t)(on0 + added) > D.T_mp && !exceeds) {
        D.exceed[list] = 1;
        told_exceed = atomicAdd(&D.ctrl->exceed_lists, 1u) + 1u;
      }
      __hip_atomic_store(&D.visible_len[list], newlen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  const uint32_t sum = last_lane(wave_running_sum(added));  // (a batch of one insertion round holds fewer than 2^32 vectors)
  if (told_exceed) D.mirror->exceed_lists = told_exceed;
  if ((threadIdx.x & (kWave - 1)) == 0 && sum) atomicAdd(&D.ctrl->ntotal, (unsigned long long)sum);
}

// The allocator's counters and the longest list are final for this batch (every block is open, and every rearrangement
// round enqueued before it has returned its spare blocks): one thread tells the host, in one store of 16 bytes.
__device__ inline void report(const Dev &D, uint32_t call_seq, uint32_t total) {
  const int32_t f = __hip_atomic_load(&D.ctrl->free_top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t in_use =
      __hip_atomic_load(&D.ctrl->cur_P, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - (uint32_t)(f > 0 ? f : 0);
  const uint32_t longest = __hip_atomic_load(&D.ctrl->max_len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *reinterpret_cast<u32x4 *>(const_cast<unsigned long long *>(&D.mirror->pool_word)) = u32x4{in_use, call_seq, total, longest};
}

__global__ __launch_bounds__(256) void k_publish(Dev D, uint32_t call_seq, uint32_t total) {
  int list = blockIdx.x * blockDim.x + threadIdx.x;
  wg_publish(D, list < D.nlist ? list : -1);
  if (list == 0) {
    report(D, call_seq, total);
    D.ctrl->fill_cur = 0u;
  }
}

// ---- a batch of up to kTailVecs vectors behind its coarse scores: one workgroup, a vector to a thread.  The vector
// that took the first new position of its list looks after the list.  What bounds an online batch is the number of
// launches (each costs the host 4 us, and the chip a start and an end) and then the chain of round trips to memory:
// reservation, opening, filling and publication as kernels of their own took 25 us per batch of 64 x 128, all of it
// the host's.  So what does not depend on the step before is asked for ahead of it: the vectors themselves, and the
// block a position falls into where that block is there already.
// splits > 0: the lists and positions are still to be had from the partial minima; 0: they are in assign and did.
// FILL: the vectors are few enough for one workgroup to move (tail_fills), and the batch is published here.
template <bool FILL>
__global__ __launch_bounds__(kTailVecs) void k_insert_tail(Dev D, int n, int splits, const double *__restrict__ pscore,
                                                           const int32_t *__restrict__ pidx,
                                                           const float *__restrict__ Y,
                                                           const int64_t *__restrict__ ids, int64_t id_base,
                                                           int32_t *__restrict__ assign, uint32_t *__restrict__ did,
                                                           uint32_t call_seq, uint32_t total) {
  __shared__ OpenShared<kTailVecs> sh;
  __shared__ uint32_t s_blk[kTailVecs], s_off[kTailVecs];  // where every vector goes (block ~0: nowhere)
  constexpr int kAhead = 4;  // chunks of the batch a thread has in registers from the start
  const int tid = threadIdx.x;
  const uint32_t T = (uint32_t)D.T_m;
  const float4 *__restrict__ y4 = reinterpret_cast<const float4 *>(Y);
  const int chunks = n * D.vchunks;
  float4 ahead[kAhead];
  if (FILL && D.storage == 0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      ahead[u] = tid + u * kTailVecs < chunks ? y4[tid + u * kTailVecs] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const uint32_t known = D.ctrl->max_len;
  const float scale = FILL && D.halves_stride ? halves_scale(D) : 1.f;
  const uint32_t inexact = FILL && D.halves_stride ? D.ctrl->half_inexact : 1u;
  int64_t id = 0;
  if (FILL && tid < n) id = ids ? ids[tid] : id_base + tid;
  int list = -1;
  uint32_t pos = 0, vis = 0, nb = 0;
  if (tid < n) {
    if (splits > 0) list = best_of_splits(D, tid, splits, pscore, pidx);
    else list = assign[tid];
    vis = D.visible_len[list];
    nb = D.nblk[list];
    if (splits > 0) pos = atomicAdd(&D.reserved_len[list], 1u);
    else pos = did[tid];
    if (!FILL && splits > 0) { assign[tid] = list; did[tid] = pos; }
  }
  const bool leads = tid < n && pos == vis;
  const uint32_t mid = pos / T;
  uint32_t blk = ~0u;
  __syncthreads();  // every position is taken
  if (FILL && tid < n && mid < nb) blk = (uint32_t)*table_entry(D, list, mid);
  const uint32_t newlen = leads ? D.reserved_len[list] : 0u;
  note_longest(D, newlen, known);
  const bool opened = wg_open<kTailVecs>(D, leads ? list : -1, nb, newlen, sh);
  if (!FILL) return;  // uniform
  if (opened) {  // uniform
    __syncthreads();
    if (tid < n && mid >= nb && mid < D.nblk[list]) blk = (uint32_t)*table_entry(D, list, mid);
  }
  if (tid < n) {
    s_blk[tid] = blk;
    s_off[tid] = pos % T;
    if (blk != ~0u) block_ids(D, blk)[pos % T] = id;
  }
  __syncthreads();
  bool exact = true;
  auto put = [&](int t, int i, int c, const float4 &v) {
    if (s_blk[i] == ~0u) return;
    block_vecs(D, s_blk[i])[vec_chunk_index(D, s_off[i], c)] = v;
    if (D.halves_stride) put_halves(D, s_blk[i], s_off[i], c, v, scale, exact);  // uniform
  };
  int t = tid;
  if (D.storage == 0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u, t += kTailVecs)
      if (t < chunks) { const int i = t / D.vchunks; put(t, i, t - i * D.vchunks, ahead[u]); }
  }
  for (; t < chunks; t += kTailVecs) {
    const int i = t / D.vchunks, c = t - i * D.vchunks;
    put(t, i, c, stored_chunk(D.storage, y4 + (size_t)i * D.d4, c));
  }
  if (!exact && !inexact) D.ctrl->half_inexact = 1u;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's part of the vectors is out ...
  __syncthreads();                                  // ... and so is everybody's before any list is published
  wg_publish(D, leads ? list : -1);
  if (tid == 0) report(D, call_seq, total);
}

// ... and the opening and the publication of a larger batch, a vector to a thread, in several workgroups (a thousand
// leaders' scattered reads and writes keep one compute unit busy for longer than a launch costs).  Whoever leads a
// list is settled by its position alone: a length that is published meanwhile lies beyond every position of the batch.
__device__ inline int led_list(const Dev &D, int n, const int32_t *__restrict__ assign, const uint32_t *__restrict__ did) {
  const int i = blockIdx.x * kBatchThreads + threadIdx.x;
  if (i >= n) return -1;
  const int list = assign[i];
  return did[i] == D.visible_len[list] ? list : -1;
}
__global__ __launch_bounds__(kBatchThreads) void k_open_batch(Dev D, int n, const int32_t *__restrict__ assign,
                                                              const uint32_t *__restrict__ did) {
  __shared__ OpenShared<kBatchThreads> sh;
  const int list = led_list(D, n, assign, did);
  const uint32_t newlen = list >= 0 ? D.reserved_len[list] : 0u;
  note_longest(D, newlen, D.ctrl->max_len);
  wg_open<kBatchThreads>(D, list, list >= 0 ? D.nblk[list] : 0u, newlen, sh);
}
__global__ __launch_bounds__(kBatchThreads) void k_publish_batch(Dev D, int n, const int32_t *__restrict__ assign,
                                                                 const uint32_t *__restrict__ did, uint32_t call_seq,
                                                                 uint32_t total) {
  wg_publish(D, led_list(D, n, assign, did));
  if (blockIdx.x == 0 && threadIdx.x == 0) report(D, call_seq, total);
}

// ---------------------------------------------------------------- launchers

void launch_reserve(const Dev &D, int64_t n, int splits, const InsertScratch &S, bool reserve,
                    int32_t *assign_out, hipStream_t s) {
  if (n <= 0) return;
  unsigned grid = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(k_reserve, dim3(grid), dim3(256), 0, s, D, n, splits, S.pscore, S.pidx,
                     reserve ? 1 : 0, assign_out ? assign_out : S.assign, S.did);
}

void launch_reserve_ordered(const Dev &D, int64_t n, const InsertScratch &S, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_reserve_ordered, dim3((unsigned)((D.nlist + 255) / 256)), dim3(256), 0, s, D, n, S.assign,
                     S.did);
}

// The partial minima of the exact coarse kernel have been read when the blocks are opened: their scratch takes the order.
static uint32_t *fill_start(const InsertScratch &S) { return reinterpret_cast<uint32_t *>(S.pidx); }
static uint2 *fill_order(const InsertScratch &S) { return reinterpret_cast<uint2 *>(S.pscore); }
// By lists pays where the moving takes longer than the launch in front of it: from 8,192 vectors, or from 2^18 chunks.
// Batches back to back, us a batch by vector / by lists: 4,096 x 32 into 4,096 lists 47.2 / 51.1, into 16,384 74.4 / 69.4, 2,048 x
// 128 into 1,024 39.4 / 41.7, 4,096 x 128 43.7 / 42.1 (into 8 lists 59.7 / 62.4), 2,048 x 768 into 8,192 75.1 / 75.9, 4,096 x 256 into
// 16,384 107.5 / 100.6, 4,096 x 768 into 8,192 122 / 115, 16,384 x 32 into 4,096 85 / 74, 65,536 x 768 into 8,192 1,377 / 1,101.
static bool fills_by_lists(const Dev &D, int64_t n, const InsertScratch &S) {
  return D.pq_m == 0 && (n >= 8192 || (n > kTailVecs && n * D.vchunks >= (int64_t)1 << 18)) &&
         (size_t)D.nlist <= S.part_cap && (size_t)n <= S.part_cap;
}

void launch_open(const Dev &D, int64_t n, const InsertScratch &S, hipStream_t s) {
  unsigned grid = (unsigned)((D.nlist + 255) / 256);
  hipLaunchKernelGGL(k_open, dim3(grid), dim3(256), 0, s, D, fills_by_lists(D, n, S) ? fill_start(S) : nullptr);
}

void launch_fill(const Dev &D, int64_t n, const float *Y, const int64_t *ids, int64_t id_base,
                 const InsertScratch &S, hipStream_t s) {
  if (n <= 0) return;
  if (fills_by_lists(D, n, S)) {
    hipLaunchKernelGGL(k_fill_order, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, D, n, ids, id_base, S.assign, S.did,
                       fill_start(S), fill_order(S));
    constexpr int64_t kTurn = kFillSlots * (int64_t)kFillXcds;
    const dim3 grid((unsigned)((n + kTurn - 1) / kTurn) * kFillXcds, (unsigned)((D.vchunks + kFillChunks - 1) / kFillChunks));
    if (D.storage == 1) hipLaunchKernelGGL(k_fill_lists<1>, grid, dim3(256), 0, s, D, n, Y, fill_order(S));
    else if (D.storage == 2) hipLaunchKernelGGL(k_fill_lists<2>, grid, dim3(256), 0, s, D, n, Y, fill_order(S));
    else hipLaunchKernelGGL(k_fill_lists<0>, grid, dim3(256), 0, s, D, n, Y, fill_order(S));
    return;
  }
  int64_t threads = n * D.vchunks;
  unsigned grid = (unsigned)((threads + 255) / 256);
  if (threads < (int64_t)1 << 31) hipLaunchKernelGGL(k_fill<uint32_t>, dim3(grid), dim3(256), 0, s, D, (uint32_t)threads, Y, ids, id_base, S.assign, S.did);
  else hipLaunchKernelGGL(k_fill<uint64_t>, dim3(grid), dim3(256), 0, s, D, (uint64_t)threads, Y, ids, id_base, S.assign, S.did);
}

// How much one workgroup moves before a launch of its own is faster, in 16-byte chunks: what its threads hold in
// registers from the start (64 x 768 floats, three times that: 25 us inside against 9 for the two launches).
constexpr int64_t kTailChunks = 4 * kTailVecs;
bool tail_fills(const Dev &D, int64_t n) { return n <= kTailVecs && D.pq_m == 0 && n * D.vchunks <= kTailChunks; }

void launch_insert_tail(const Dev &D, int64_t n, int splits, const float *Y, const int64_t *ids, int64_t id_base,
                        const InsertScratch &S, uint32_t call_seq, uint32_t total, hipStream_t s) {
  const dim3 batch((unsigned)((n + kBatchThreads - 1) / kBatchThreads));
  if (tail_fills(D, n))
    hipLaunchKernelGGL(k_insert_tail<true>, dim3(1), dim3(kTailVecs), 0, s, D, (int)n, splits, S.pscore, S.pidx, Y, ids,
                       id_base, S.assign, S.did, call_seq, total);
  else if (splits > 0)
    hipLaunchKernelGGL(k_insert_tail<false>, dim3(1), dim3(kTailVecs), 0, s, D, (int)n, splits, S.pscore, S.pidx, Y,
                       ids, id_base, S.assign, S.did, call_seq, total);
  else
    hipLaunchKernelGGL(k_open_batch, batch, dim3(kBatchThreads), 0, s, D, (int)n, S.assign, S.did);
}

void launch_publish_batch(const Dev &D, int64_t n, const InsertScratch &S, uint32_t call_seq, uint32_t total, hipStream_t s) {
  const dim3 batch((unsigned)((n + kBatchThreads - 1) / kBatchThreads));
  hipLaunchKernelGGL(k_publish_batch, batch, dim3(kBatchThreads), 0, s, D, (int)n, S.assign, S.did, call_seq, total);
}

void launch_publish(const Dev &D, uint32_t call_seq, uint32_t total, hipStream_t s) {
  unsigned grid = (unsigned)((D.nlist + 255) / 256);
  hipLaunchKernelGGL(k_publish, dim3(grid), dim3(256), 0, s, D, call_seq, total);
}

}  // namespace rtams
