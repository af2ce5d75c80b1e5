/*
 * rtams_measure.h - measurement aids of librtams.so.  NOT part of the method (arXiv 2408.02937) and not
 * needed to use the index: the benchmark and the profiling runs call them to time the list-scan kernel
 * inside a request and to calibrate hardware counters against kernels of known traffic.
 * Conventions as in rtams.h: d_* are device pointers, hip_stream is a hipStream_t passed as void*,
 * every function returns RTAMS_OK or a negative rtams_status.
 */
#ifndef RTAMS_MEASURE_H
#define RTAMS_MEASURE_H

#include "rtams.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Measured duration of the list-scan kernel: with the parameter "profile_scan"
 * set to 1, every search brackets its scan launch with two HIP events on the
 * caller's stream; this call adds up the pairs of the requests that have
 * finished (ms_sum in milliseconds, launches = how many) and optionally resets
 * the sums.  Does not synchronise. */
int rtams_scan_time(rtams_index *ix, double *ms_sum, int64_t *launches, int reset);
/* Which kernel those timed launches were: launches3[0] counts the scans of the
 * vector unit (k_scan), [1] those on the matrix cores (k_scan_mm), [2] those
 * over product-quantiser codes (k_pq_scan), each since the last reset, counted
 * at launch while "profile_scan" is 1.  The library chooses per request. */
int rtams_scan_kernels(rtams_index *ix, int64_t *launches3, int reset);
/* ... and how many were scans of the halves beside float lists (k_scan_halves), which are none of those three. */
int rtams_scans_of_halves(rtams_index *ix, int64_t *launches, int reset);
/* What the last request on a stream resource left in its scratch (0 .. n_resources - 1; n_resources is the static
 * array of rtams_search_noalloc, which the next request of any index overwrites), for tests of how requests are
 * answered.  Per query of its nq: h_bounds the pruning bound as the key the scan compared with (0xFFFFFFFF: every
 * candidate kept), h_kept the number of candidates the scan kept.  *path, how it was scanned: 0 by the vector unit from
 * a plan, 1 by the vector unit without one ("small_requests"), 2 by the matrix cores in floats, 3 by their 16-bit
 * instructions, 4 over product-quantiser codes, 5 by the halves beside the lists.  Any pointer may be NULL.  The caller has waited for the request. */
int rtams_request_trace(rtams_index *ix, int32_t resource, int64_t nq, uint32_t *h_bounds, uint32_t *h_kept,
                        int32_t *path);
/* A plain device-to-device copy kernel
 * (bytes a multiple of 16).  Profiler counters of HBM traffic are scaled by
 * what they read for this kernel, whose traffic is known. */
int rtams_copy_plain(void *d_dst, const void *d_src, size_t bytes, void *hip_stream);
/* A kernel that only reads `bytes`
 * (a multiple of 16) of device memory; d_sink points to 4 bytes of device
 * memory it may write.  Its rate is the practical ceiling a streaming read
 * reaches on the chip, reported beside the list scan's. */
int rtams_read_plain(const void *d_src, size_t bytes, float *d_sink, void *hip_stream);
#ifdef __cplusplus
}
#endif
#endif /* RTAMS_MEASURE_H */
