// The list scan of flat lists on the matrix cores.
#include "scan_tile.h"

namespace rtams {

// The scores of a tile are a small dense contraction (vectors x queries over the dimensions), and the
// interleaved layout hands a wavefront exactly the operand the 4x4x1 matrix instruction wants: lane =
// vector, one coordinate per instruction (search_common.h).  A workgroup takes one work item (list,
// segment, tile of up to 32 of the queries probing the list).  The tile's queries go to LDS once, in
// groups of four (rows past the tile's last query are zero), each with the words the scan needs of
// it: how far its list goes, its bound, where its survivor records go.  Then the four wavefronts share
// out the segment's groups of 64 vectors and work on their own: per chunk of 4 dimensions a wavefront
// loads 1 KiB ONCE, lane l reads the float4 of query 4 g + l % 4 of every group of queries g, and four
// matrix instructions per group of queries use them up.  Per 1 KiB of list data that is 4 matrix
// instructions of 8 cycles for every 4 queries, against 16 to 32 vector instructions of 4 cycles, and
// the vector unit is left with |x|^2 (squared distances only): the kernel sits on the memory side,
// and a list is read once per 32 of the queries that probe it.
// Inner products are returned as the contraction leaves them (the bound's sample uses the same
// instruction sequence, so a pair scores the same bits there and here).  Squared distances take the
// norm form |x|^2 + |q|^2 - 2 <x, q>, whose rounding errors scale with the norms: the bound they are
// compared with was loosened by the proven margin, and the selection scores its finalists again in
// the direct form, so what is returned is exactly what the direct form gives.
// Afterwards lane l holds, for each group of queries g, the scores of vectors 4 (l / 4) .. + 3 against
// ONE query, 4 g + l % 4.  What is not worse than that query's bound goes to a staging area of the
// wavefront in LDS (places from ballots, no waiting); when the area is full, and when the wavefront
// is through with its groups, the staged survivors are counted per query with LDS atomics, ONE
// global atomic instruction reserves the places of all the tile's queries, and the records go out.
// (A returning global atomic per group of queries and of vectors, waited for each time, cost more
// than the scan itself: dozens of wavefronts reserve from the same few counters.)

// The groups g_lo + wave, g_lo + wave + 4, ... below g_hi of the list against QG groups of four queries.
// first_b: the block that holds the wavefront's first group (looked up by the caller).
// ST: what the lists keep.  A 16-byte chunk of halves or bytes is widened in registers, one float4 of coordinates at a
// time, each against the matching float4 of the queries: the conversions run beside the matrix instructions, where
// the vector-unit kernel has them in front of its own arithmetic (256 queries x 32 probes over 1 M x 128 bytes: 114 us
// there, bound by instruction issue, for 129 MB of lists).
template <int METRIC, int QG, int ST>
__device__ __forceinline__ void scan_groups_mm(const Dev &D, const SearchScratch &S, int list, uint32_t g_lo,
                                               uint32_t g_hi, uint32_t first_b, const float4 *qs,
                                               const TileQuery *tq, WaveStage &st) {
  constexpr int kPrefetch = 4;  // chunks per register set: 8 KiB of loads in flight per wavefront
  constexpr int kPieces = pieces_of(ST);
  const int vc = D.vchunks;
  const int qstride = D.d4 + 1;  // float4s between two queries in LDS: an odd stride keeps the four rows a read touches on different banks
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 3;
  const float4 *__restrict__ qrow = qs + sub * qstride;  // query `sub` of group 0; group g is 4 g rows on
  const uint32_t gpb = (uint32_t)D.groups_per_block;
  const size_t group_stride = (size_t)vc * kWave;
  Staging stage{S, tq, st, 0u};
  // The wavefront's groups of vectors as a software pipeline ACROSS the groups: while one is being
  // streamed the block number of the next is looked up, and the first loads of the next go out before
  // the survivors of this one are dealt with, so that neither the two dependent table reads nor the
  // first trip to memory of a group stand between two groups (a quarter of a group's time at d = 128).
  const int d4_main = vc & ~(2 * kPrefetch - 1);  // chunks that go through the two register sets
  float4 sa[kPrefetch], sb[kPrefetch];
  auto load_set = [&](float4 *s, const float4 *__restrict__ p, int cb) {
#pragma unroll
    for (int u = 0; u < kPrefetch; ++u) s[u] = p[(size_t)(cb + u) * kWave];
    __builtin_amdgcn_sched_barrier(0);  // loads are issued here, not sunk towards their use
  };
  auto place = [&](uint32_t g, uint32_t b) -> const float4 * {
    return block_vecs(D, b) + (size_t)(g % gpb) * group_stride + lane;
  };
  uint32_t g0 = g_lo + (uint32_t)wave;
  if (g0 >= g_hi) return;  // nothing staged yet
  first_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)first_b);
  const float4 *x = place(g0, first_b);
  uint32_t cur_b = first_b;  // the block of group g0 (the same for every lane, as is all that follows from it: scalar registers)
  if (d4_main) load_set(sa, x, 0);
  for (;;) {
    const uint32_t g_next = g0 + kMmWaves;
    const bool more = g_next < g_hi;  // uniform over the wavefront
    uint32_t next_b = 0;
    if (more) next_b = (uint32_t)*table_entry(D, list, g_next / gpb);  // on its way while this group is streamed
    MfmaAcc acc[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) acc[g] = (MfmaAcc){0.f, 0.f, 0.f, 0.f};
    float nrm = 0.f;  // |x|^2 of the lane's own vector
    // every accumulator takes the coordinates in their order; the chains of the groups of queries are
    // interleaved so that no instruction waits for the one in front of it
    auto use = [&](const float4 &v, int c) {
      if (METRIC == 0) accumulate<1>(nrm, v, v);
      constexpr int kHalf = QG == 6 ? 3 : QG > 4 ? 4 : QG;  // groups of queries whose coordinates are held at once (a divisor of QG)
#pragma unroll
      for (int h = 0; h < QG; h += kHalf) {
        float4 y[kHalf];
#pragma unroll
        for (int g = 0; g < kHalf; ++g) y[g] = qrow[4 * (h + g) * qstride + c];
#pragma unroll
        for (int g = 0; g < kHalf; ++g) mfma_step(acc[h + g], v.x, y[g].x);
#pragma unroll
        for (int g = 0; g < kHalf; ++g) mfma_step(acc[h + g], v.y, y[g].y);
#pragma unroll
        for (int g = 0; g < kHalf; ++g) mfma_step(acc[h + g], v.z, y[g].z);
#pragma unroll
        for (int g = 0; g < kHalf; ++g) mfma_step(acc[h + g], v.w, y[g].w);
      }
    };
    auto use_chunk = [&](const float4 &raw, int c) {
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
        use(chunk_piece<ST>(raw, p), c * kPieces + p);
        if (kPieces > 1) __builtin_amdgcn_sched_barrier(0);  // one piece's widened values at a time
      }
    };
    auto use_set = [&](const float4 *s, int cb) {
#pragma unroll
      for (int u = 0; u < kPrefetch; ++u) use_chunk(s[u], cb + u);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (d4_main) {  // set a holds chunks 0 .. kPrefetch - 1 of this group already
      int c = 0;
#pragma unroll 1
      for (; c + 2 * kPrefetch < d4_main; c += 2 * kPrefetch) {
        load_set(sb, x, c + kPrefetch);
        use_set(sa, c);
        load_set(sa, x, c + 2 * kPrefetch);
        use_set(sb, c + kPrefetch);
      }
      load_set(sb, x, c + kPrefetch);
      use_set(sa, c);
      use_set(sb, c + kPrefetch);
    }
    for (int c = d4_main; c < vc; ++c) use_chunk(x[(size_t)c * kWave], c);
    const float4 *x_next = x;
    if (more) {  // the next group's first loads go out before this group's survivors are dealt with
      next_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)next_b);
      x_next = place(g_next, next_b);
      if (d4_main) load_set(sa, x_next, 0);
    }

    // scores -> keys; which of the lane's 4 candidates per group of queries survive
    auto norm_of = [&](int r) {  // of candidate r (moved again for every group of queries: four registers kept for it were spilled)
      return r == 0 ? quad_broadcast<0>(nrm) : r == 1 ? quad_broadcast<1>(nrm) : r == 2 ? quad_broadcast<2>(nrm) : quad_broadcast<3>(nrm);
    };
    const uint32_t vbase = g0 * kWave + 4u * (uint32_t)(lane >> 2);
    const uint32_t slot_base = slot_of(D, cur_b, (g0 % gpb) * kWave + 4u * (uint32_t)(lane >> 2));
#pragma unroll
    for (int g = 0; g < QG; ++g) {
      const TileQuery me = tq[4 * g + sub];  // len 0 for rows past the tile: nothing of theirs is kept
      uint32_t key[4], pass = 0u;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float sc = acc[g][r];
        // (an infinite coordinate makes the norm form inf - inf: such a vector is infinitely far, as the direct form has it)
        sc = METRIC == 0 ? fminf(fmaf(-2.f, sc, norm_of(r) + me.qn), __builtin_inff()) : -sc;
        key[r] = key_of_float(sc + 0.0f);
        if (vbase + r < me.len && key[r] <= me.bound) pass |= 1u << r;
      }
      stage.keep(pass, key, slot_base, (uint32_t)(4 * g + sub));
    }
    if (!more) break;
    g0 = g_next;
    x = x_next;
    cur_b = next_b;
  }
  if (stage.staged) stage.flush();
}

// ---- squared distances to lists of halves and bytes.  What is stored is an operand of the 16-bit matrix instructions as it
// is (halves), or a byte's conversion away (bf16 holds them exactly); the query, 24 bits of each coordinate, is split into
// three pieces of the operand's type once per tile, and the products of the pieces, which are exact, add up in 32 bits to
// the product of the query.  v_mfma_f32_16x16x32: lane l supplies eight coordinates of vector (or query) l % 16, and the 16
// bytes that the lists keep of a vector are such eight, or twice such eight: four chunks of 16 vectors are the operand of
// one or two instructions, whatever coordinate falls to which place, as long as both operands agree.  Queries whose second
// and third pieces are zero (byte values) leave them out.
// Against 4x4x1 instructions on widened floats (d x 8 clocks for every 4 queries and 64 vectors, and a conversion per
// coordinate beside them) this takes d x 6 clocks for 16 queries, or d x 2: 256 queries x 32 probes over 1 M x 128 bytes,
// 1,024 lists, 87 us with the former and 56 with these.  Where it pays: narrow_scan_pays.
// The first piece is summed for itself, so that the norm form keeps its margin (norm_form_slack); |x|^2 is a sum of integers for bytes, and for halves the diagonal of the vectors' products with
// themselves.  The selection scores its finalists again in the direct form, as behind the other scan.
typedef _Float16 HalfX8 __attribute__((ext_vector_type(8)));
typedef __bf16 Bf16X8 __attribute__((ext_vector_type(8)));
template <int ST>
__device__ __forceinline__ MfmaAcc narrow_product(const u32x4 &a, const u32x4 &b, const MfmaAcc &acc) {
  if (ST == 1) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(HalfX8, a), __builtin_bit_cast(HalfX8, b), acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(Bf16X8, a), __builtin_bit_cast(Bf16X8, b), acc, 0, 0, 0);
}
// eight bytes as eight bf16
__device__ __forceinline__ u32x4 bytes_to_bf16(uint32_t lo, uint32_t hi) {
  u32x4 out;
  auto two = [](float a, float b) {  // the upper halves of two floats
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  };
  out[0] = two((float)(lo & 255u), (float)((lo >> 8) & 255u));
  out[1] = two((float)((lo >> 16) & 255u), (float)(lo >> 24));
  out[2] = two((float)(hi & 255u), (float)((hi >> 8) & 255u));
  out[3] = two((float)((hi >> 16) & 255u), (float)(hi >> 24));
  return out;
}
// Row of query pieces in LDS: the coordinates of whole fours of chunks, and 16 bytes that spread the rows over the banks.
constexpr int kNarrowPieces = 3;

// Groups g_lo + wave, ... below g_hi against 16 CB queries.  qp: [pieces][rows][row_bytes].
template <int ST, int CB>
__device__ __forceinline__ void scan_groups_narrow(const Dev &D, const SearchScratch &S, int list, uint32_t g_lo, uint32_t g_hi,
                                                   uint32_t first_b, const char *qp, int rows, int pieces, const TileQuery *tq,
                                                   WaveStage &st) {
  constexpr int kSteps = ST == 2 ? 2 : 1;  // instructions to a chunk
  const int vc = D.vchunks, quads = (vc + 3) / 4;
  const uint32_t row_bytes = narrow_row_bytes(D), piece_bytes = row_bytes * (uint32_t)rows;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int col = lane & 15, kg = lane >> 4;  // the lane's vector of 16 and query of 16, and its chunk of four
  const uint32_t gpb = (uint32_t)D.groups_per_block;
  const size_t group_stride = (size_t)vc * kWave;
  const char *my_q = qp + (uint32_t)col * row_bytes + (uint32_t)kg * (kSteps * 16u);
  Staging stage{S, tq, st, 0u};
  uint32_t g0 = g_lo + (uint32_t)wave;
  if (g0 >= g_hi) return;  // nothing staged yet
  uint32_t cur_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)first_b);
  auto place = [&](uint32_t g, uint32_t b) {
    return reinterpret_cast<const u32x4 *>(block_vecs(D, b)) + (size_t)(g % gpb) * group_stride;
  };
  u32x4 cur[4];
  auto load = [&](u32x4 *to, const u32x4 *x, int quad) {  // the lane's chunk of the quad, of its vector in each block of 16
    const uint32_t at = (uint32_t)(min(4 * quad + kg, vc - 1) * kWave + col);
#pragma unroll
    for (int b = 0; b < 4; ++b) to[b] = x[at + 16u * b];
    __builtin_amdgcn_sched_barrier(0);  // the loads go out here
  };
  const u32x4 *x = place(g0, cur_b);
  load(cur, x, 0);
  for (;;) {
    const uint32_t g_next = g0 + kMmWaves;
    const bool more = g_next < g_hi;  // uniform over the wavefront
    uint32_t next_b = 0;
    if (more) next_b = (uint32_t)*table_entry(D, list, g_next / gpb);  // on its way while this group is streamed
    MfmaAcc acc[4][CB], low[4][CB], gram[ST == 1 ? 4 : 1];
    uint32_t sq[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[b][cb] = low[b][cb] = (MfmaAcc){0.f, 0.f, 0.f, 0.f};
      if (ST == 1) gram[b] = (MfmaAcc){0.f, 0.f, 0.f, 0.f};
    }
    const u32x4 *x_next = x;
#pragma unroll 1
    for (int quad = 0; quad < quads; ++quad) {
      u32x4 nxt[4];
      if (quad + 1 < quads) {
        load(nxt, x, quad + 1);
      } else if (more) {  // the next group's first loads go out before this group's survivors are dealt with
        next_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)next_b);
        x_next = place(g_next, next_b);
        load(nxt, x_next, 0);
      }
      if (4 * quad + kg >= vc) {  // chunks past the vector
#pragma unroll
        for (int b = 0; b < 4; ++b) cur[b] = (u32x4){0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int j = 0; j < kSteps; ++j) {
        u32x4 a[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (ST == 1) {
            a[b] = cur[b];
            gram[b] = narrow_product<ST>(a[b], a[b], gram[b]);
          } else {
            const uint32_t w0 = cur[b][2 * j], w1 = cur[b][2 * j + 1];
            sq[b] = __builtin_amdgcn_udot4(w0, w0, sq[b], false);
            sq[b] = __builtin_amdgcn_udot4(w1, w1, sq[b], false);
            a[b] = bytes_to_bf16(w0, w1);
          }
        }
        auto add_piece = [&](int pc, MfmaAcc (&to)[4][CB]) {
          u32x4 y[CB];
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            y[cb] = *reinterpret_cast<const u32x4 *>(my_q + (uint32_t)pc * piece_bytes + (uint32_t)(16 * cb) * row_bytes + (uint32_t)quad * (4u * kSteps * 16u) + 16u * j);
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int b = 0; b < 4; ++b) to[b][cb] = narrow_product<ST>(a[b], y[cb], to[b][cb]);
        };
        add_piece(0, acc);
#pragma unroll 1
        for (int pc = 1; pc < pieces; ++pc) add_piece(pc, low);  // uniform
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) cur[b] = nxt[b];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[b][cb][r] += low[b][cb][r];
    __builtin_amdgcn_sched_barrier(0);  // (the second sums' registers are free from here on)
    // (what the lane's place comes to below is worked out here again, not kept in registers through the loop above)
    int kge = kg, cole = col;
    asm volatile("" : "+v"(kge), "+v"(cole));
    // |x|^2 of the lane's four rows of a block: rows 4 kg .. 4 kg + 3 (the result's layout)
    float nr[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (ST == 2) {
        uint32_t t = sq[b] + (uint32_t)__shfl_xor((int)sq[b], 16);
        t += (uint32_t)__shfl_xor((int)t, 32);
#pragma unroll
        for (int r = 0; r < 4; ++r) nr[b][r] = (float)(uint32_t)__shfl((int)t, 4 * kge + r);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) nr[b][r] = __shfl(gram[b][r], 16 * kge + 4 * kge + r);  // the diagonal: column 4 kge + r of those rows
      }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const TileQuery me = tq[16 * cb + cole];  // len 0 for rows past the tile: nothing of theirs is kept
      const float m2 = -2.f * me.unscale;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t vbase = g0 * kWave + 16u * b + 4u * (uint32_t)kge;
        uint32_t key[4], pass = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // (an infinite coordinate makes the norm form inf - inf: such a vector is infinitely far, as the direct form has it)
          const float sc = fminf(fmaf(m2, acc[b][cb][r], nr[b][r] + me.qn), __builtin_inff());
          key[r] = key_of_float(sc + 0.0f);
          if (vbase + r < me.len && key[r] <= me.bound) pass |= 1u << r;
        }
        stage.keep(pass, key, slot_of(D, cur_b, (g0 % gpb) * kWave + 16u * b + 4u * (uint32_t)kge), (uint32_t)(16 * cb + cole));
      }
    }
    if (!more) break;
    g0 = g_next;
    x = x_next;
    cur_b = next_b;
  }
  if (stage.staged) stage.flush();
}

// Wavefronts to a SIMD: four where the launch is short and its last workgroups count (256 queries x 32 probes over 1 M x
// 128, 2,048 items: bytes 89 us with three and 87 with four, floats 105 and 104: what is scanned comes from memory at
// 7 TB/s meanwhile, and only the launch's end is shorter); three for long scans and inner products of floats, which
// gain nothing by it.  Squared distances to floats, requests of 64 to 256 queries with four against three: 32 to 80
// dimensions 0.94 to 1.02 of the time (0.98 on average), 128 to 256 0.99 to 1.02 (1.01), 512 and more 0.99 to 1.01.
template <int METRIC, bool STEAL, int ST, bool NARROW>
__global__ __launch_bounds__(kMmWaves *kWave, STEAL || NARROW || (METRIC == 1 && ST == 0) ? 3 : 4) void k_scan_mm(Dev D, int max_nprobe, const float *__restrict__ Q,
                                                             SearchScratch S, int tile_rows) {
  // [tile_rows][d / 4 + 1] coordinates of the tile's queries (or the pieces of narrow lists), [tile_rows] TileQuery, [wavefronts] WaveStage
  extern __shared__ float4 lds_mm[];
  uint4 desc;
  uint32_t seg;
  const uint32_t pairs = take_item<STEAL>(S, desc, seg);
  if (pairs == 0) return;  // uniform over the workgroup
  const int list = __builtin_amdgcn_readfirstlane((int)desc.x);  // (one item to the workgroup)
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.y);
  const int d4 = D.d4, qstride = d4 + 1;
  float4 *qs = lds_mm;
  const uint32_t row_bytes = NARROW ? narrow_row_bytes(D) : 0u;
  TileQuery *tq = reinterpret_cast<TileQuery *>(NARROW ? reinterpret_cast<float4 *>(reinterpret_cast<char *>(lds_mm) + (size_t)kNarrowPieces * tile_rows * row_bytes)
                                                       : lds_mm + (size_t)tile_rows * qstride);
  WaveStage &st = reinterpret_cast<WaveStage *>(tq + tile_rows)[threadIdx.x / kWave];
  // groups of four queries of this tile: 1, 2, 3, 4, 6 or 8, whichever holds the item's queries; exactly
  // that many rows of LDS are set up, and the instantiation below reads exactly that many (the plan never
  // puts more queries into a tile than tile_rows)
  int qg = (int)((pairs + 3u) / 4u);
  qg = qg == 5 ? 6 : qg == 7 ? 8 : qg;
  const int rows = NARROW ? (pairs > 16u ? 32 : 16) : 4 * qg;
  if (rows > tile_rows || rows > kMmTileMax) return;  // a descriptor the launch was not sized for: nothing is scanned
  // The block number of the wavefront's first group of vectors is asked for now (two dependent reads)
  // and used after the tile is set up.  Never past the list's chain, whatever the descriptors say.
  const uint32_t g_begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)desc.w) * seg;
  const uint32_t g_have = D.nblk[list] * (uint32_t)D.groups_per_block;
  uint32_t first_b = 0;
  {
    const uint32_t g0 = g_begin + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (g0 < g_have) first_b = (uint32_t)*table_entry(D, list, g0 / (uint32_t)D.groups_per_block);
  }
  // the tile's queries: words first (one thread per row), then coordinates (the workgroup together)
  uint32_t my_len = 0;
  if ((int)threadIdx.x < rows) {
    TileQuery t{};
    if (threadIdx.x < pairs) {
      const uint32_t pk = S.grouped[first + threadIdx.x];
      t.q = pk >> 10;
      const size_t o = (size_t)t.q * max_nprobe + (pk & 1023u);
      t.len = S.probe_len[o];
      const unsigned long long qb = S.qbase[t.q];
      t.keys = (uint64_t)(uintptr_t)rec_keys_of(S, qb);
      t.poss = (uint64_t)(uintptr_t)rec_poss_of(S, qb);
      t.bound = S.bound[t.q];
      if (METRIC == 0) t.qn = S.qnorm[t.q];
      if (NARROW) t.unscale = ST == 1 ? 1.f / half_piece_scale(t.qn) : 1.f;
    }
    tq[threadIdx.x] = t;
    my_len = t.len;
  }
  __shared__ uint32_t s_pieces[kMmWaves];
  if (NARROW) {
    // ... as pieces; coordinates past d are zero
    const int cols = (int)((row_bytes - 16u) / 8u), total = rows * cols;  // four coordinates at a time
    char *qp = reinterpret_cast<char *>(lds_mm);
    const uint32_t piece_bytes = row_bytes * (uint32_t)rows;
    uint32_t have = 0u;
    constexpr int kInFlight = 4, kThreads = kMmWaves * kWave;
    for (int base = (int)threadIdx.x; base < total; base += kInFlight * kThreads) {
      float4 v[kInFlight];
      float qn[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int idx = base + u * kThreads, row = idx < total ? idx / cols : rows, col = idx - row * cols;
        const bool on = row < (int)pairs && col < d4;
        const uint32_t q = on ? S.grouped[first + row] >> 10 : 0u;
        v[u] = on ? reinterpret_cast<const float4 *>(Q + (size_t)q * D.d)[col] : make_float4(0.f, 0.f, 0.f, 0.f);
        qn[u] = on && ST == 1 ? S.qnorm[q] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int idx = base + u * kThreads, row = idx < total ? idx / cols : rows, col = idx - row * cols;
        if (row >= rows) continue;
        const float scale = ST == 1 ? half_piece_scale(qn[u]) : 1.f;
        float w[4] = {v[u].x * scale, v[u].y * scale, v[u].z * scale, v[u].w * scale};
#pragma unroll
        for (int pc = 0; pc < kNarrowPieces; ++pc) {
          uint32_t bits[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (ST == 1) {
              const _Float16 h = (_Float16)w[e];
              bits[e] = (uint32_t)__builtin_bit_cast(uint16_t, h);
              w[e] -= (float)h;
            } else {
              bits[e] = __float_as_uint(w[e]) >> 16;
              w[e] -= __uint_as_float(bits[e] << 16);
            }
            if (bits[e] & 0x7fffu) have = max(have, (uint32_t)pc + 1u);
          }
          *reinterpret_cast<uint2 *>(qp + (size_t)pc * piece_bytes + (size_t)row * row_bytes + (size_t)col * 8) =
              make_uint2(bits[0] | bits[1] << 16, bits[2] | bits[3] << 16);
        }
      }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) have = max(have, (uint32_t)__shfl_xor((int)have, o));
    if ((threadIdx.x & (kWave - 1)) == 0) s_pieces[threadIdx.x / kWave] = have;
  } else
  // coordinates: the rows x d / 4 float4s of the tile are dealt out over the workgroup, eight independent
  // loads per thread in flight (a row at a time would be a chain of memory latencies per row); which
  // query a row holds is read from the grouped pairs again rather than waited for in LDS
  {
    const int total = rows * d4;
    constexpr int kInFlight = 8, kThreads = kMmWaves * kWave;
    for (int base = (int)threadIdx.x; base < total; base += kInFlight * kThreads) {
      uint32_t pk[kInFlight];
      int row[kInFlight], col[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int idx = base + u * kThreads;
        row[u] = idx < total ? idx / d4 : rows;
        col[u] = idx - row[u] * d4;
        pk[u] = row[u] < (int)pairs ? S.grouped[first + row[u]] : 0u;
      }
      float4 v[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u)
        v[u] = row[u] < (int)pairs ? reinterpret_cast<const float4 *>(Q + (size_t)(pk[u] >> 10) * D.d)[col[u]]
                                   : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < kInFlight; ++u)
        if (row[u] < rows) qs[row[u] * qstride + col[u]] = v[u];
    }
  }
  // how far the longest of the tile's snapshots goes (the first wavefront holds the lengths)
  __shared__ uint32_t s_maxlen;
  if (threadIdx.x < kWave) {
    uint32_t m = my_len;
    for (int o = kWave / 2; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
    if (threadIdx.x == 0) s_maxlen = m;
  }
  __syncthreads();
  uint32_t g_end = (s_maxlen + kWave - 1) / kWave;  // groups any query of the tile wants
  if (g_end > g_begin + seg) g_end = g_begin + seg;  // ... inside this item's segment
  if (g_end > g_have) g_end = g_have;
  // no barrier from here on: the wavefronts only read the tile
  if (NARROW) {
    const char *qp = reinterpret_cast<const char *>(lds_mm);
    const int pieces = __builtin_amdgcn_readfirstlane((int)max(max(s_pieces[0], s_pieces[1]), max(s_pieces[2], s_pieces[3])));
    if (rows == 16) scan_groups_narrow<ST, 1>(D, S, list, g_begin, g_end, first_b, qp, rows, pieces, tq, st);
    else scan_groups_narrow<ST, 2>(D, S, list, g_begin, g_end, first_b, qp, rows, pieces, tq, st);
    return;
  }
  switch (qg) {
    case 1: scan_groups_mm<METRIC, 1, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
    case 2: scan_groups_mm<METRIC, 2, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
    case 3: scan_groups_mm<METRIC, 3, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
    case 4: scan_groups_mm<METRIC, 4, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
    case 6: scan_groups_mm<METRIC, 6, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
    default: scan_groups_mm<METRIC, 8, ST>(D, S, list, g_begin, g_end, first_b, qs, tq, st); break;
  }
}

typedef void (*MmKernel)(Dev, int, const float *, SearchScratch, int);
static const MmKernel mm_kernels[2][2][3] = {
    {{k_scan_mm<0, false, 0, false>, k_scan_mm<0, false, 1, false>, k_scan_mm<0, false, 2, false>},
     {k_scan_mm<0, true, 0, false>, k_scan_mm<0, true, 1, false>, k_scan_mm<0, true, 2, false>}},
    {{k_scan_mm<1, false, 0, false>, k_scan_mm<1, false, 1, false>, k_scan_mm<1, false, 2, false>},
     {k_scan_mm<1, true, 0, false>, k_scan_mm<1, true, 1, false>, k_scan_mm<1, true, 2, false>}}};
static const MmKernel mm_narrow[2][2] = {{k_scan_mm<0, false, 1, true>, k_scan_mm<0, false, 2, true>},
                                         {k_scan_mm<0, true, 1, true>, k_scan_mm<0, true, 2, true>}};

hipError_t allow_large_lds_scan_mm() {  // (wide vectors only)
  hipError_t e = hipSuccess;
  for (int i = 0; i < 16 && e == hipSuccess; ++i)
    e = allow_lds(i < 12 ? mm_kernels[i / 6][i / 3 % 2][i % 3] : mm_narrow[(i - 12) / 2][i % 2], kMmLdsMax);
  return e;
}

void launch_scan_mm(const Dev &D, const ScanShape &sh, int max_nprobe, const float *Q, const SearchScratch &S,
                    hipStream_t s) {
  const MmKernel kernel = scans_narrow(D) ? mm_narrow[D.scan_steal ? 1 : 0][D.storage - 1] : mm_kernels[D.metric][D.scan_steal ? 1 : 0][D.storage];
  hipLaunchKernelGGL(kernel, dim3((unsigned)sh.grid), dim3((unsigned)sh.threads),
                     sh.lds, s, D, max_nprobe, Q, S, sh.tile_q);
}

}  // namespace rtams
