/*
 * dq8 -- calls of dq8.h with scratch memory of the caller's.  Conventions, arguments and results are those of the calls
 * they are named after.
 */
#ifndef DQ8_WORKSPACE_H
#define DQ8_WORKSPACE_H

#include "dq8.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Scratch memory.  Compression that reads x twice has to merge the maxima of the first pass.  With scratch memory the first
 * pass leaves one maximum per workgroup there and the second combines them; without, the scales are cleared and merged with
 * atomics, which is one launch more.  The codes and scales are the same.
 * dq8_workspace_bytes: what dq8_encode_ws can use for these arguments, 0 when it needs none (host arithmetic).
 * dq8_encode_ws: dq8_encode with `workspace_bytes` bytes of device memory at `workspace`, 4-byte aligned, whose contents are of
 * no meaning before and after; it must not overlap the other arrays, and calls that may run at the same time must not share
 * it.  Where the call is captured into a graph, the memory is the graph's for as long as that may be replayed.  NULL or too few
 * bytes: as dq8_encode.
 */
size_t dq8_workspace_bytes(size_t n, size_t block, unsigned flags);
int dq8_encode_ws(int kind, const float *x, size_t n, size_t block, float *scales, uint8_t *codes,
                  unsigned flags, void *workspace, size_t workspace_bytes, void *hip_stream);

/* dq8_encode_segments with scratch memory, see dq8_encode_ws. */
size_t dq8_workspace_bytes_segments(size_t n, size_t n_seg, unsigned flags);
int dq8_encode_segments_ws(int kind, const float *x, size_t n, const uint64_t *bounds, size_t n_seg, float *scales,
                           uint8_t *codes, unsigned flags, void *workspace, size_t workspace_bytes, void *hip_stream);

/* dq8_error_stats with scratch memory, 8-byte aligned here: the statistics of a long array that is one block then
 * go there by workgroup and are added in a fixed order, so that the sums do not differ between calls. */
size_t dq8_workspace_bytes_stats(size_t n, size_t block, unsigned flags);
int dq8_error_stats_ws(int kind, const float *x, size_t n, size_t block, float *scales, unsigned flags, double *stats,
                       double *means, void *workspace, size_t workspace_bytes, void *hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* DQ8_WORKSPACE_H */
