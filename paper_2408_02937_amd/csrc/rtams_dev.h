// Device-side view of the pool: layout constants, block format, block table.
// Internal to the library; nothing here is part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rtams {

constexpr int kWave = 64;            // gfx950 wavefront
constexpr int kHeaderBytes = 128;    // block header, padded so ids and vectors stay line aligned
constexpr int kTableBase = 32;       // entries of a list's first block-table segment
constexpr int kTableSegs = 20;       // segment s holds kTableBase << s entries
constexpr int kMaxK = 1024;
constexpr int kMaxNprobe = 1024;

// Header of a memory block ("mh" of the paper: previous / next header and block
// info), followed inside the block by the id list "ml" and the vectors "mv".
struct BlockHeader {
  int32_t prev;      // physical block before this one in the chain, -1 at the head
  int32_t next;      // physical block after this one, -1 at the tail
  int32_t owner;     // list that owns the block, -1 when free
  int32_t seq;       // position in the owner's chain
  int32_t capacity;  // T_m
  int32_t size;      // vectors visible in this block
  int32_t pad[26];
};
static_assert(sizeof(BlockHeader) == kHeaderBytes, "header size");

// What the matrix-core filter knows of the centroids (coarse_mfma.hip): magnitudes as float bits, all of them of the
// centroids less their mean; norms of the scaled halves.
struct CentroidStats {
  uint32_t top_bits;   // largest coordinate
  uint32_t norm_bits;  // largest norm, scaled
  uint32_t res_bits;   // largest norm of what the halves leave out, scaled
  uint32_t bias_bits;  // largest |bias|
  float mean_norm;     // norm of the mean
  uint32_t bad;        // some coordinate is not finite, or too large for its square
};

// Control words shared by all kernels (one cache line each for the hot ones).
struct Ctrl {
  uint32_t cur_P;            // bump pointer of the central pool
  uint32_t pad0[31];
  int32_t free_top;          // number of entries on the free stack
  uint32_t pad1[31];
  uint32_t slab_cur;         // bump pointer of the block-table slab
  uint32_t pad2[31];
  int32_t error;             // sticky rtams_status raised by a kernel
  uint32_t exceed_lists;     // lists for which Exceed() holds
  unsigned long long ntotal; // vectors visible
  uint32_t max_len;          // longest list, taken where a batch's blocks are opened (a batch dropped for lack of blocks counts)
  int32_t search_error;      // rtams_status raised by a kernel of a search (scratch too small): inserts do not look at it
  CentroidStats cen;
  uint32_t fill_cur;         // vectors of the batch whose lists have their place in the order of the fill (0 between batches)
  uint32_t half_top;         // largest coordinate of a centroid, float bits ...
  float half_scale;          // ... and the power of two that the halves beside the lists are scaled by
  uint32_t half_inexact;     // some vector's halves are not its floats
  uint32_t pad3[16];
};

// Words the device writes straight into pinned host memory, so the host can
// read them without synchronising.
struct HostMirror {
  volatile int32_t error;
  volatile uint32_t exceed_lists;
  volatile int32_t search_error;
  volatile uint32_t halves_failed;  // a query's scan of halves left more than halves are for (select.hip); the host clears it
  volatile uint32_t rearr_state;  // of the last rearrangement round: 0 done, 1 another round owed, 2 stalled for lack of a spare block
  // The two words below are written by every publication, by one thread in one store of 16 bytes; the host reads either
  // of them whole.  pool_word: (number of the last insertion call published << 32) | blocks in use after it.  The host
  // takes from it how many blocks are left without waiting for the data stream.
  alignas(16) volatile unsigned long long pool_word;
  // (length of the longest list << 32) | vectors handed to add up to this batch, modulo 2^32: with what the host has
  // handed over since, a bound of any list at any time.
  volatile unsigned long long len_word;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Dev {
  int32_t d, nlist, metric, T_m;
  int32_t pq_m;             // 0: flat lists; M > 0: product-quantiser codes, M bytes per vector
  int32_t scan_mfma;        // flat lists: the scan's dot products run on the matrix cores, 2: on the 16-bit instructions (set per request)
  int32_t scan_single;      // a request of few groups of vectors in short lists: the vector-unit scan takes them one at a time (set per request)
  int32_t scan_steal;       // a long scan on the matrix cores: XCDs that are done take items of the others (set per request)
  int32_t scan_min_choice;  // shortest segment the plan may choose, as a power of two of pairs of groups (-1: the kernel's default; set per request)
  int32_t scan_byte_weight; // cost of reading a group of a list, in queries' worth of arithmetic (0: the default; set per request)
  int32_t d4;               // d / 4
  int32_t storage;          // what flat lists keep of a coordinate: 0 float, 1 half, 2 byte
  int32_t vchunks;          // 16-byte chunks of a stored vector: d / 4, d / 8 or d / 16
  int32_t groups_per_block; // T_m / 64
  uint32_t nblocks;         // |P|
  uint32_t slab_cap;        // entries in the table slab
  int64_t T_mp;             // rearrangement threshold
  uint64_t block_stride;    // bytes
  uint32_t ids_off;         // byte offset of the id list inside a block
  uint32_t vec_off;         // byte offset of the vectors inside a block
  char *blocks;
  Ctrl *ctrl;
  HostMirror *mirror;       // pinned host memory, device-visible
  float *centroids;         // [nlist][d]
  float *centroids_t;       // the same numbers as [d / 4][nlist] chunks of 4 coordinates: chunk j of consecutive centroids side by side
  float *cmean;             // [d] mean of the centroids
  float *cbias;             // [nlist] the part of an approximate coarse score that only the centroid decides
  u32x4 *chalf;             // [nlist] the centroids less their mean as halves (layout: coarse_mfma.hip)
  int32_t dgroups;          // groups of 8 coordinates of a row of halves, padded with zeros to whole steps of 32 coordinates: 4 ceil(d / 32)
  float *codebooks;         // [pq_m][256][d / pq_m] (product-quantised lists only)
  float *codebooks_t;       // the same with the entries innermost: [pq_m][d / pq_m][256] (for coding inserted vectors)
  uint32_t *reserved_len;   // [nlist] next free position (atomicAdd target)
  uint32_t *visible_len;    // [nlist] length searches may read
  uint32_t *online;         // [nlist] vectors since the last rearrangement
  uint32_t *nblk;           // [nlist] blocks in the chain
  uint8_t *exceed;          // [nlist] Exceed() holds
  int32_t *seg_dir;         // [nlist][kTableSegs] slab offset of each table segment, -1 unset
  int32_t *slab;            // block-table entries
  int32_t *free_stack;      // [nblocks]
  int32_t *mark;            // [nblocks] scratch for validation
  // (behind all that the kernels of small requests read)
  char *halves;             // flat lists of floats: the halves of block b's vectors, at b * halves_stride
  uint64_t halves_stride;   // bytes of a block's halves (0: none are kept)
  int32_t hchunks;          // 16-byte chunks of a vector's halves: d / 8, rounded up
  int32_t scan_halves;      // the request reads them: 1, 2 with tiles of 32 queries (set per request)
};

// ---- block table: a growable array per list, made of doubling segments ----
__host__ __device__ inline int table_seg(uint32_t i) {
  uint32_t v = i / kTableBase + 1;
#if defined(__HIP_DEVICE_COMPILE__)
  return 31 - __clz((int)v);
#else
  int s = 0;
  while (v >>= 1) ++s;
  return s;
#endif
}
__host__ __device__ inline uint32_t table_seg_first(int s) {
  return (uint32_t)kTableBase * ((1u << s) - 1u);
}

__device__ inline int32_t *table_entry(const Dev &D, int list, uint32_t i) {
  int s = table_seg(i);
  int32_t off = D.seg_dir[(size_t)list * kTableSegs + s];
  return D.slab + off + (i - table_seg_first(s));
}
// The same in its two dependent steps, for callers that want the first on its way early: where the
// table segment of entry i starts (the word exists for every list and segment), then the entry
// (which exists only below the list's number of blocks).
__device__ inline int32_t table_dir(const Dev &D, int list, uint32_t i) {
  return D.seg_dir[(size_t)list * kTableSegs + table_seg(i)];
}
__device__ inline int32_t *table_entry_at(const Dev &D, int32_t dir, uint32_t i) {
  return D.slab + dir + (i - table_seg_first(table_seg(i)));
}

// A vector's place in the pool as one 32-bit number (block * T_m + place in the block; the pool holds
// at most 2^32 places, which rtams_create checks): what a search keeps of a surviving candidate, so
// that whoever needs its id or its coordinates later goes straight to the block.  The block stays
// what it was until the request has finished: a rearrangement waits for the requests in flight
// before it reuses a block.
__device__ inline uint32_t slot_of(const Dev &D, uint32_t b, uint32_t place) { return b * (uint32_t)D.T_m + place; }

__device__ inline BlockHeader *block_header(const Dev &D, uint32_t b) {
  return reinterpret_cast<BlockHeader *>(D.blocks + (size_t)b * D.block_stride);
}
__device__ inline int64_t *block_ids(const Dev &D, uint32_t b) {
  return reinterpret_cast<int64_t *>(D.blocks + (size_t)b * D.block_stride + D.ids_off);
}
__device__ inline float4 *block_vecs(const Dev &D, uint32_t b) {
  return reinterpret_cast<float4 *>(D.blocks + (size_t)b * D.block_stride + D.vec_off);
}

// Product-quantised lists keep the same shape with 4 codes (one 32-bit word) as the chunk:
// word index of codes 4c..4c+3 of the vector at offset moff.
__device__ inline uint32_t *block_codes(const Dev &D, uint32_t b) {
  return reinterpret_cast<uint32_t *>(D.blocks + (size_t)b * D.block_stride + D.vec_off);
}
__device__ inline size_t code_word_index(const Dev &D, uint32_t moff, int c) {
  uint32_t group = moff / kWave, lane = moff % kWave;
  return ((size_t)group * (D.pq_m / 4) + c) * kWave + lane;
}

// Interleaved vector layout inside a block (the paper's equation for "mv",
// re-derived for 64-wide wavefronts): vectors are taken in groups of 64; inside
// a group, chunk c (16 bytes: dimensions 4c..4c+3 of floats, 8c..8c+7 of halves,
// 16c..16c+15 of bytes) of the 64 vectors is contiguous, one float4 per vector.
// A wavefront reading chunk c of a group loads 1 KiB of consecutive memory,
// lane = vector.
__device__ inline size_t vec_chunk_index(const Dev &D, uint32_t moff, int c) {
  uint32_t group = moff / kWave, lane = moff % kWave;
  return ((size_t)group * D.vchunks + c) * kWave + lane;
}

// ---- copies straight from memory to LDS: lane l of the wavefront brings the 16 bytes at src + 16 l, and the 1 KiB lies in
// order at the LDS address `to` (both the same for every lane; lane16 = 16 l).  The compiler does not know of them: whoever
// asks for copies waits for them (the wavefront's count of loads, in front of the barrier that hands them to others),
// and does not end before they have come.
__device__ __forceinline__ void copy_to_lds(const void *src, uint32_t to, uint32_t lane16) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(to), "v"(lane16), "s"(src) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

// ---- sums, smallest and largest over a wavefront, by moves between its lanes inside the vector unit (data-parallel
// primitives: rows of 16 lanes, then the last lane of a row to the next one, and of the first two rows to the last two).  A
// __shfl is a trip to LDS, some 60 clocks of a chain; a step here is one or two instructions.  The chains of a request are full of
// them (a radix selection has two such reductions and a running sum for every pass): 10 queries over 10,000 x 32 floats 31.4 us a
// request with shuffles and 29.6 with these, one over 1 M x 128 45.1 and 42.7, 256 over codes of 16 bytes 116.2 and 113.0.  wave_step<I>: the value of the I-th step's lane, or `old` where
// that step brings none.
template <int I>
__device__ __forceinline__ uint32_t wave_step(uint32_t old, uint32_t v) {
  constexpr int kCtrl = I == 0 ? 0x111 : I == 1 ? 0x112 : I == 2 ? 0x114 : I == 3 ? 0x118 : I == 4 ? 0x142 : 0x143;
  constexpr int kRows = I == 4 ? 0xa : I == 5 ? 0xc : 0xf;
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, kCtrl, kRows, 0xf, false);
}
template <int I>
__device__ __forceinline__ unsigned long long wave_step(unsigned long long old, unsigned long long v) {
  return (unsigned long long)wave_step<I>((uint32_t)old, (uint32_t)v) |
         (unsigned long long)wave_step<I>((uint32_t)(old >> 32), (uint32_t)(v >> 32)) << 32;
}
template <int I>
__device__ __forceinline__ double wave_step(double old, double v) {
  return __longlong_as_double((long long)wave_step<I>((unsigned long long)__double_as_longlong(old), (unsigned long long)__double_as_longlong(v)));
}
// lane l: the sum of lanes 0 .. l
template <typename T>
__device__ __forceinline__ T wave_running_sum(T v) {
  v += wave_step<0>((T)0, v); v += wave_step<1>((T)0, v); v += wave_step<2>((T)0, v);
  v += wave_step<3>((T)0, v); v += wave_step<4>((T)0, v); v += wave_step<5>((T)0, v);
  return v;
}
// in the last lane: `pick` (associative, commutative, pick(a, a) = a) over all lanes
template <typename T, typename Pick>
__device__ __forceinline__ T wave_reduce_last(T v, Pick pick) {
  v = pick(v, wave_step<0>(v, v)); v = pick(v, wave_step<1>(v, v)); v = pick(v, wave_step<2>(v, v));
  v = pick(v, wave_step<3>(v, v)); v = pick(v, wave_step<4>(v, v)); v = pick(v, wave_step<5>(v, v));
  return v;
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1); }
__device__ __forceinline__ unsigned long long last_lane(unsigned long long v) {
  return (unsigned long long)last_lane((uint32_t)v) | (unsigned long long)last_lane((uint32_t)(v >> 32)) << 32;
}
// the other lane of a pair, of a pair of pairs: l ^ 1, l ^ 2
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), X == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}
// in every lane: the sum over the S lanes (a power of two, at most a wavefront) of its group
__device__ __forceinline__ uint32_t group_sum(uint32_t v, int S) {
  if (S > 1) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);   // l ^ 1
  if (S > 2) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);   // l ^ 2
  if (S > 4) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true);  // the other four of eight (mirrored: they agree)
  if (S > 8) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, true);  // the other eight of sixteen
  if (S > 16) v += (uint32_t)__shfl_xor((int)v, 16);
  if (S > 32) v += (uint32_t)__shfl_xor((int)v, 32);
  return v;
}

// ---- narrow storage: a 16-byte chunk holds 8 halves or 16 bytes.  piece s of a chunk is the
// float4 of its dimensions 4s..4s+3 (2 pieces of halves, 4 of bytes).
typedef _Float16 Half2 __attribute__((ext_vector_type(2)));
template <int ST>
__device__ __forceinline__ float4 chunk_piece(const float4 &raw, int s) {
  if (ST == 1) {
    const Half2 a = __builtin_bit_cast(Half2, s == 0 ? raw.x : raw.z);
    const Half2 b = __builtin_bit_cast(Half2, s == 0 ? raw.y : raw.w);
    return make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
  } else if (ST == 2) {
    const uint32_t w = __float_as_uint(s == 0 ? raw.x : s == 1 ? raw.y : s == 2 ? raw.z : raw.w);
    return make_float4((float)(w & 255u), (float)((w >> 8) & 255u), (float)((w >> 16) & 255u), (float)(w >> 24));
  }
  return raw;
}
constexpr int pieces_of(int storage) { return storage == 1 ? 2 : storage == 2 ? 4 : 1; }
// the conversions on the way in: IEEE round to nearest even (overflow to infinity) for halves;
// nearest integer, ties to even, clamped to 0..255 for bytes (fmaxf drops a NaN)
__device__ __forceinline__ uint32_t pack_halves(float lo, float hi) {
  Half2 h;
  h.x = (_Float16)lo;
  h.y = (_Float16)hi;
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ uint32_t byte_of(float f) { return (uint32_t)fminf(fmaxf(__builtin_rintf(f), 0.f), 255.f); }
__device__ __forceinline__ uint32_t pack_bytes(const float4 &v) {
  return byte_of(v.x) | (byte_of(v.y) << 8) | (byte_of(v.z) << 16) | (byte_of(v.w) << 24);
}

// ---- halves beside the lists of floats: every coordinate under one power-of-two scale as a half.  A scan that reads them instead
// of the floats has half the bytes to read; what it keeps is scored again from the floats, so they decide nothing but what
// is looked at.  The scale brings the largest coordinate of a centroid to 2^8: vectors may be 2^7 times as large before a half
// overflows.  In groups of 64 vectors as the lists, but within a group 32 coordinates (four 16-byte chunks) of a vector side by
// side, vector after vector, then the next 32; what is left of d (rounded up to 8, with zeros) likewise.  So what is written of a
// vector is whole 64-byte pieces, and 16 vectors' worth of a matrix instruction is 1 KiB in one run.
__device__ inline float halves_scale(const Dev &D) { return D.ctrl->half_scale; }
__device__ inline float halves_scale_for(uint32_t t) {  // t: that coordinate, float bits
  if (t < 0x00800000u || t >= 0x7f800000u) return 1.f;
  int s = 8 - ((int)(t >> 23) - 127);
  s = s > 100 ? 100 : s < -100 ? -100 : s;
  return __uint_as_float((uint32_t)(s + 127) << 23);
}
// (what lies below the smallest normal half is zero, whatever a unit makes of subnormals)
__device__ __forceinline__ float no_subnormal_half(float x) { return fabsf(x) < 6.1035156e-5f ? 0.f : x; }
// (halves times one over the scale are the floats, to the last bit: `exact` stays true.  The floats themselves are asked, not what
// the scale makes of them, which may be zero where they are not; one over it, a power of two, is made of its bits.  Comparing the
// scaled coordinates, and all of them with zero, cost a load of 500,000 x 768 3 %.)
__device__ __forceinline__ uint2 pack_four_halves(const float4 &v, float scale, bool &exact) {
  const float a = v.x * scale, b = v.y * scale, c = v.z * scale, e = v.w * scale;
  const uint2 h = make_uint2(pack_halves(no_subnormal_half(a), no_subnormal_half(b)), pack_halves(no_subnormal_half(c), no_subnormal_half(e)));
  const Half2 lo = __builtin_bit_cast(Half2, h.x), hi = __builtin_bit_cast(Half2, h.y);
  const float inv = __uint_as_float(0x7F000000u - __float_as_uint(scale));
  exact = exact && (float)lo.x * inv == v.x && (float)lo.y * inv == v.y && (float)hi.x * inv == v.z && (float)hi.y * inv == v.w &&
          fmaxf(fmaxf(fabsf(a), fabsf(b)), fmaxf(fabsf(c), fabsf(e))) < 65536.f;
  return h;
}
__device__ inline char *block_halves(const Dev &D, uint32_t b) { return D.halves + (size_t)b * D.halves_stride; }
// byte offset, inside a block's halves, of 16-byte chunk c of the vector at moff
__device__ inline size_t half_chunk_at(const Dev &D, uint32_t moff, uint32_t c) {
  const uint32_t quad = c / 4u, width = min((uint32_t)D.hchunks - 4u * quad, 4u);
  return (size_t)(moff / kWave) * ((size_t)D.hchunks * (kWave * 16u)) + (size_t)quad * (kWave * 64u) + (moff % kWave * width + c % 4u) * 16u;
}
// chunk c of four floats of the vector at moff
__device__ __forceinline__ void put_halves(const Dev &D, uint32_t b, uint32_t moff, int c, const float4 &v, float scale, bool &exact) {
  const uint2 h = pack_four_halves(v, scale, exact);
  char *to = block_halves(D, b) + half_chunk_at(D, moff, (uint32_t)c >> 1);
  if (c == D.d4 - 1 && !(c & 1)) *reinterpret_cast<u32x4 *>(to) = u32x4{h.x, h.y, 0u, 0u};
  else reinterpret_cast<uint2 *>(to)[c & 1] = h;
}

}  // namespace rtams
