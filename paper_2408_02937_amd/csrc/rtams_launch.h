// Host-callable launchers of the kernels, one translation unit per group.
// Internal to the library.
#pragma once
#include "rtams_dev.h"

namespace rtams {

// Work items of the scan of one request.  The items are ordered by list; each
// XCD owns a contiguous range of them.
struct ScanQueues {
  uint32_t begin[9];    // XCD x owns items begin[x] .. begin[x+1]-1
  uint32_t seg_groups;  // 64-vector groups per work item
  // Long scans on the matrix cores: an XCD that has run out of its own items takes items of the others
  // from the back of their ranges (all of these words are zero when the request starts).
  uint32_t back[8];     // items taken from the back of XCD y's range so far
  uint32_t done_mask;   // bit y: nothing is left to take from XCD y
  uint32_t pad[13];
};
static_assert(sizeof(ScanQueues) == 32 * 4, "the request's clearing pass covers the queue words");

// The scan keeps, for every query, only the candidates that are not worse than
// the query's BOUND (the k-th best score of a sample of its candidates, set
// before the scan starts): they are appended to the query's survivor records.

// Per-request scratch of one stream resource (device pointers into its slice).
struct SearchScratch {
  double *scores;       // [max_batch][nlist] coarse scores in the fixed double arithmetic
  float *approx;        // [max_batch][nlist] approximate coarse scores from the matrix cores
  int32_t *probe_list;  // [max_batch][max_nprobe]
  uint32_t *probe_len;  // [max_batch][max_nprobe] list lengths as seen by this request
  unsigned long long *qbase;  // [max_batch] start of the query's slice of rec_key / rec_pos
  uint32_t *qtotal;     // [max_batch] candidates of the query
  uint32_t *bound;      // [max_batch] key of the score the scan compares with
  float *qnorm;         // [max_batch] squared norms of the queries (norm form of the squared distance)
  u32x4 *qhalf;         // the queries as halves for the matrix-core coarse scores, then their RowMeta (coarse_mfma.hip)
  uint32_t *done_count; // [max_batch] workgroups of a query that are done with their part of it (small.hip, bound.h; 0 between requests)
  uint32_t *rec_cnt;    // survivors recorded so far, of query q at rec_cnt[q << rec_shift] (rec_count())
  int rec_shift;
  unsigned long long *cursor; // bump pointer into the survivor records
  uint32_t *list_cnt;   // [nlist] queries probing each list
  uint32_t *pair_start; // [nlist] where the pairs of a probed list start in `grouped`
  uint32_t *pair_slot;  // [max_batch][max_nprobe] rank of the pair among the pairs of its list
  uint32_t *grouped;    // [max_batch * max_nprobe] pairs (query << 10 | probe) grouped by list
  uint4 *plist;         // [min(nlist, max_batch * max_nprobe)] per probed list, in list order: {list, unused, pairs,
                        // length as seen by the grouping step}
  uint4 *tile_desc;     // [item_cap] {list, first pair of the tile, pairs of the tile, segment} per item (scans of halves: half_item_word() for the pairs)
  uint32_t item_cap;
  ScanQueues *queues;   // work items of this request, split into one queue per XCD
  float *lut;           // [max_batch][pq_m][256] sub-scores of the queries against the codebooks (PQ lists)
  uint32_t *rec_key;    // survivors: key of the score (smaller is better) ...
  uint32_t *rec_pos;    // ... and its place in the pool (slot_of)
  unsigned long long cand_cap;  // entries of each of the two arrays
  // The reserve shared by all resources, cut into chunks of equal size.  A request whose queries do not
  // all fit into the slice leases ONE chunk (the first query in need takes it, the others share it);
  // queries placed there carry bit 63 in their qbase; the request's last selection workgroup returns it.
  uint32_t *ovf_leased;         // [ovf_chunks] central: 0 free, 1 leased
  uint32_t ovf_chunks;
  unsigned long long ovf_chunk_cap;  // entries of a chunk (in each of the two arrays)
  uint32_t *ovf_key, *ovf_pos;  // central: [ovf_chunks * ovf_chunk_cap] each
  uint32_t *req_chunk;          // this resource's request: 0 none, 1 + the chunk it holds
  uint32_t *req_done;           // selection workgroups of the request that have finished
  unsigned long long *req_cursor;  // entries of the chunk handed out to the request's queries
};

constexpr unsigned long long kInOverflow = 1ull << 63;  // flag in SearchScratch::qbase
constexpr int kMaxOverflowChunks = 32;

constexpr int kScanTileQueries = 8;  // queries that share one pass over a list

// What the matrix-core filter knows of a vector: the factor that turns an accumulated product into a score, and
// the band, twice the error bound of an approximate score (both in coarse_mfma.hip).
struct RowMeta {
  float scale, band;
};

// What a tile of approximate coarse scores is reduced to, per row: the tile's smallest score and the columns within the
// error band of it, up to eight; of a tile that has more, every column is scored exactly for that row.  24 bytes: a
// kept score is 8 bits, how many 255ths of the band it lies above the smallest (it only has to say whether the column is
// a candidate, and erring low by a step costs a candidate in a few hundred).  With four columns and whole scores, 40
// bytes, data whose clusters hold tens of centroids each had such a tile in a quarter of its rows: 131,072 x 256 against
// 8,192 centroids in 100 clusters took 5.0 ms and takes 1.8 (2.5 with the three products of bf16 pairs that the one of
// halves replaced); centroids spread evenly 1.20 ms before and 1.16 now.
constexpr int kTileCands = 8;
struct TileCands {
  int32_t tiles;   // tiles per row = ceil(nlist / width)
  int32_t width;   // centroids of a tile, 256 or 128 (chosen per launch)
  int64_t rows;    // rows the arrays hold with tiles of 256
  float *tmin;     // [rows][tiles]
  uint32_t *cnt;   // [rows][tiles] columns within the band (may exceed kTileCands)
  uint16_t *kept;  // [rows][tiles][kTileCands] steps above tmin << 8 | column of the tile
};

// Scratch of the insertion path (lives in the pool's control region).
struct InsertScratch {
  int32_t *assign;   // [max_add_batch] list of each vector
  uint32_t *did;     // [max_add_batch] position inside the list
  double *pscore;    // [part_cap] best score per (vector, centroid split)
  int32_t *pidx;     // [part_cap]
  size_t part_cap;
  TileCands tiles;   // per (row, tile of centroids) digest of the approximate scores of one sub-round
  u32x4 *yhalf;      // [tile_rows] the vectors of one sub-round as halves
  RowMeta *ymeta;    // [tile_rows] their scales and bands
  int64_t tile_rows; // rows one sub-round may hold
};

// Scratch of one rearrangement round (lives in the pool's control region).
struct RearrangeHead {
  int32_t list;    // list being rearranged, -1 none
  uint32_t count;  // moves of this round
  uint32_t nvict;  // occupants that had to be moved out of the way
  uint32_t done;   // the round reaches the end of the chain
  uint32_t state;  // after the round: 0 the list is contiguous (or nothing was to do), 1 another round is owed,
                   // 2 stalled: no spare block in the pool
  uint32_t cursor; // where the search for the next exceeding list starts (kept from round to round)
};
struct RearrangeScratch {
  RearrangeHead *head;
  uint32_t cap;        // moves per round
  uint32_t *mv_t;      // [cap] chain position of each move, ascending
  uint32_t *kind;      // [cap] what sits at the target: 0 never handed out, 1 free, 2 a block in use
  uint32_t *vic_rank;  // [cap] rank among the occupants in use
  uint32_t *vic_new;   // [cap] block the occupant is copied to
  uint32_t *old_src;   // [cap] block the list gives up
  int32_t *vic_list;   // [cap] owner of the occupant
  int32_t *vic_seq;    // [cap] its position in the owner's chain
};

// A kernel whose workgroups may take more than 64 KiB of LDS has to be told so, on every device by itself: rtams_create
// does it for the index's.
hipError_t allow_large_lds_coarse();
hipError_t allow_large_lds_dots();
hipError_t allow_large_lds_group();
hipError_t allow_large_lds_scan_mm();
hipError_t allow_large_lds_pq_scan();
hipError_t allow_large_lds_scan_halves();
template <typename Kernel>
inline hipError_t allow_lds(Kernel kernel, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// coarse.hip ---------------------------------------------------------------
int coarse_vt(int d);                      // vectors per workgroup for this dimension
int coarse_splits(const Dev &D, int64_t n, size_t part_cap);
int coarse_vectors(const Dev &D, int64_t n);  // vectors of a workgroup's tile for this batch
// full score matrix scores[n][nlist]
void launch_coarse_scores(const Dev &D, int64_t n, const float *Y, double *scores,
                          unsigned long long *cursor_to_clear, uint32_t *zero, int zero_n, hipStream_t s);
// per (vector, split) best centroid
void launch_coarse_argmin(const Dev &D, int64_t n, const float *Y, int splits, double *pscore,
                          int32_t *pidx, hipStream_t s);

// coarse_mfma.hip ------------------------------------------------------------
constexpr int kTailVecs = 1024;  // vectors of an insertion batch that one workgroup sees to behind the coarse scores (insert.hip)
// When the matrix-core filter runs in front of the exact coarse arithmetic: the
// batch has to be a dense contraction large enough to repay the extra kernel and
// the refinement (measured crossover on MI355X, d = 128 and 768: about 1 M (query,
// centroid) pairs for a search).
inline bool mfma_pays_for_search(int64_t nq, int64_t nlist) { return nq >= 32 && nq * nlist >= (int64_t)1 << 20; }
// An assignment pays from 2^19 pairs and 2^26 coordinates of them.  Below that the filter is a few workgroups, each a
// chain of d / 32 steps, in front of a refinement and a tail that no longer fuse.  From 1,024 vectors it pays from 2^18
// pairs, and above that number, where the tail does not fuse either way, from 2^25 coordinates.
// Insertion batches back to back, vectors of which several centroids are candidates, exact / filter in us: d 768, 256 x
// 1,024 47 / 60, x 2,048 65 / 61, 64 x 4,096 44 / 55, x 8,192 66 / 57, 1,024 x 256 62 / 66, x 420 93 / 67;  d 256, 256 x
// 1,024 32 / 35, x 2,048 40 / 36, 2,048 x 128 53 / 41;  d 128, 128 x 2,048 24 / 31, x 4,096 30 / 32, x 8,192 39 / 33, 512 x
// 1,024 34 / 36;  d 32, 128 x 8,192 26 / 30, 256 x 8,192 40 / 32, 1,024 x 1,024 30 / 37, 3,700 x 160 37 / 40, x 300 47 / 38,
// 1,100 x 1,024 36 / 36;  d 1536, 256 x 1,024 72 / 90, x 2,048 98 / 92.
inline bool mfma_pays_for_assign(int64_t m, int64_t nlist, int64_t d) {
  return m >= 32 && m * nlist >= (int64_t)1 << (m >= 1024 ? 18 : 19) && m * nlist * d >= (int64_t)1 << (m > kTailVecs ? 25 : 26);
}
// 16-byte units the halves of `rows` rows take: whole blocks of 16 rows
__host__ __device__ inline size_t half_units(int64_t rows, int dgroups) { return (size_t)((rows + 15) / 16 * 16) * dgroups; }
// a request's RowMeta behind the halves of its n queries (32 of them at least: the room is 32 dgroups bytes a query)
__host__ __device__ inline RowMeta *search_row_meta(const Dev &D, int64_t n, u32x4 *half) {
  return reinterpret_cast<RowMeta *>(half + half_units(n, D.dgroups));
}
void launch_centroid_halves(const Dev &D, hipStream_t s);  // behind the transposed copy
void launch_centroid_transpose(const Dev &D, hipStream_t s);  // the copy the exact coarse kernel streams
// (`half` takes the n rows as halves, half_units(n, dgroups) units)
void launch_coarse_mfma(const Dev &D, int64_t n, const float *Y, u32x4 *half, float *approx,
                        unsigned long long *cursor_to_clear, uint32_t *zero, int zero_n, hipStream_t s);
void launch_coarse_tiles(const Dev &D, int64_t n, const float *Y, u32x4 *half, RowMeta *meta, TileCands &tc,
                         hipStream_t s);  // chooses tc.width and tc.tiles
void launch_assign_refine(const Dev &D, int64_t n, const float *Y, const RowMeta *meta, const TileCands &tc, bool reserve,
                          int32_t *assign, uint32_t *did, hipStream_t s);

// insert.hip -----------------------------------------------------------------
void launch_reserve(const Dev &D, int64_t n, int splits, const InsertScratch &S, bool reserve,
                    int32_t *assign_out, hipStream_t s);
// Positions for a batch whose lists are already in S.assign, in the order of the batch (one thread per list).
void launch_reserve_ordered(const Dev &D, int64_t n, const InsertScratch &S, hipStream_t s);
void launch_open(const Dev &D, int64_t n, const InsertScratch &S, hipStream_t s);
void launch_fill(const Dev &D, int64_t n, const float *Y, const int64_t *ids, int64_t id_base,
                 const InsertScratch &S, hipStream_t s);
// (publications report to the host under the call's number and with `total`, the vectors handed to add so far)
void launch_publish(const Dev &D, uint32_t call_seq, uint32_t total, hipStream_t s);
// A batch of at most kTailVecs vectors: reservation (splits > 0: from the partial minima; 0: done), opening and,
// where tail_fills() says so, filling and publication; otherwise a fill and launch_publish_batch follow.
bool tail_fills(const Dev &D, int64_t n);
void launch_insert_tail(const Dev &D, int64_t n, int splits, const float *Y, const int64_t *ids, int64_t id_base,
                        const InsertScratch &S, uint32_t call_seq, uint32_t total, hipStream_t s);
void launch_publish_batch(const Dev &D, int64_t n, const InsertScratch &S, uint32_t call_seq, uint32_t total, hipStream_t s);

// probe.hip, group.hip, scan.hip, pq_scan.hip, select.hip ---------------------
void launch_probe_plan(const Dev &D, int64_t nq, int nprobe, int max_nprobe, const SearchScratch &S,
                       const float *Q, bool from_approx, int32_t *probe_out, hipStream_t s);
// One launch does three things side by side: one workgroup cuts the scan into work
// items, one groups the pairs by list, one per query sets the query's bound.
// (Quantised lists are scanned per query: only the bounds are set.)
void launch_group(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int k, const float *Q,
                  int item_budget, const SearchScratch &S, hipStream_t s);
void launch_scan(const Dev &D, int64_t nq, int nprobe, int max_nprobe, const float *Q, int item_budget,
                 const SearchScratch &S, hipStream_t s);
// the scan of flat float lists on the matrix cores (launch_scan hands such requests on to it)
struct ScanShape;
void launch_scan_mm(const Dev &D, const ScanShape &sh, int max_nprobe, const float *Q, const SearchScratch &S,
                    hipStream_t s);
// the scan of the halves beside float lists (launch_scan hands such requests on to it)
void launch_scan_halves(const Dev &D, const ScanShape &sh, int max_nprobe, const SearchScratch &S, hipStream_t s);
// the scan over product-quantiser codes (launch_scan hands quantised lists on to it)
void launch_pq_scan(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int item_budget,
                    const SearchScratch &S, hipStream_t s);
// a small request over flat lists (small.hip): coarse scores, probes and bounds; then the scan, `units` (of one or two groups)
// at most to a query's lists as far as the host knows; launch_select follows
constexpr double kSmallBytes = 32e6;
bool small_request(const Dev &D, int64_t nq, int nprobe, int64_t avg_len, int64_t longest);
void launch_small_front(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int k, const float *Q, const SearchScratch &S,
                        hipStream_t s);
void launch_scan_small(const Dev &D, int64_t nq, int nprobe, int max_nprobe, int64_t units, const float *Q,
                       const SearchScratch &S, hipStream_t s);
void launch_select(const Dev &D, int64_t nq, int k, const float *Q, const SearchScratch &S, float *out_dist, int64_t *out_ids,
                   hipStream_t s);

// pq.hip -----------------------------------------------------------------------
void launch_pq_fill(const Dev &D, int64_t n, const float *Y, const int64_t *ids, int64_t id_base,
                    const InsertScratch &S, hipStream_t s);
void launch_pq_transpose(const Dev &D, hipStream_t s);  // after the codebooks changed
void launch_pq_export(const Dev &D, int list, int64_t n, int64_t *ids, uint8_t *codes, hipStream_t s);

// rearrange.hip --------------------------------------------------------------
void launch_rearr_plan(const Dev &D, const RearrangeScratch &R, int list, hipStream_t s);
void launch_rearr_step(const Dev &D, const RearrangeScratch &R, int phase, hipStream_t s);
void launch_rearr_release(const Dev &D, const RearrangeScratch &R, hipStream_t s);

// maint.hip ------------------------------------------------------------------
void launch_export(const Dev &D, int list, int64_t n, int64_t *ids, float *vecs, hipStream_t s);
void launch_chain_copy(const Dev &D, int list, int32_t *out, hipStream_t s);
void launch_list_info(const Dev &D, int list, int32_t *out4, hipStream_t s);
void launch_validate(const Dev &D, int32_t *result2, hipStream_t s);
void launch_copy_plain(void *dst, const void *src, size_t bytes, hipStream_t s);
void launch_read_plain(const void *src, size_t bytes, float *sink, hipStream_t s);

}  // namespace rtams
