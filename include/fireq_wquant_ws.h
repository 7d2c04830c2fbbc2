/*
 * fireq_wquant_ws.h -- two calls of the offline weight quantiser of fireq.h with device scratch.
 *
 * fq_cas_scales_ws and fq_pts_exponent_ws are fq_cas_scales and fq_pts_exponent (same operands, checks and status codes)
 * with fq_cas_scales_workspace_bytes(N,K) / fq_pts_exponent_workspace_bytes(N,K) bytes of device memory, 16-byte aligned
 * (FQ_ERR_ALIGN; FQ_ERR_MEMORY if smaller; where that size is 0, or with workspace == NULL, the call is the one without
 * scratch).  With it the rows of a large matrix are shared out over the chip and the workgroups' partial results folded,
 * in a fixed order, by a second kernel.
 *
 * fq_pts_exponent_ws gives the result of fq_pts_exponent: its statistics are minima and maxima.
 * fq_cas_scales_ws adds the same FP64 terms as fq_cas_scales in another order, which follows from N, K and the number of the
 * device's compute units (a W that is not 16-byte aligned takes the call without scratch).  On one device lambda is the
 * same from call to call.  It is that of fq_cas_scales, bit for bit, wherever a channel's sum of magnitudes is exact in FP64
 * -- it stays below 2^46 times the largest power of two in the channel's smallest non-zero magnitude, as weights' sums do --
 * and at most one FP32 step from it elsewhere.
 *
 * The scratch may be reused or freed once the work enqueued by the call has finished; calls that overlap in time need
 * scratch of their own.
 */
#ifndef FIREQ_WQUANT_WS_H
#define FIREQ_WQUANT_WS_H

#include "fireq.h"

#ifdef __cplusplus
extern "C" {
#endif

size_t fq_cas_scales_workspace_bytes(int N, int K);
int fq_cas_scales_ws(const uint16_t *W_bf16, float target, float *lambda, int N, int K,
                     void *workspace, size_t workspace_bytes, void *stream);
size_t fq_pts_exponent_workspace_bytes(int N, int K);
int fq_pts_exponent_ws(const uint16_t *W_bf16, const float *lambda, int *n_out, int N, int K,
                       void *workspace, size_t workspace_bytes, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* FIREQ_WQUANT_WS_H */
