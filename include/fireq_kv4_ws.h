/*
 * fireq_kv4_ws.h -- the attention output product of fireq.h with device scratch.
 *
 * fq_kv4_output_ws is fq_kv4_output (same operands, checks and status codes) with
 * fq_kv4_output_workspace_bytes(H,R,T) bytes of device memory, 16-byte aligned (FQ_ERR_ALIGN; FQ_ERR_MEMORY if
 * smaller; where that size is 0, or with workspace == NULL, the call is fq_kv4_output).  With it, few heads with long
 * caches are cut into token slices, so that the product covers the chip, and a second kernel adds the slices' FP32 sums
 * in a fixed order: the last bits differ from those of the unsliced sum, and are the same from call to call.
 * The scratch may be reused or freed once the work enqueued by the call has finished; calls that overlap in time
 * need scratch of their own.
 */
#ifndef FIREQ_KV4_WS_H
#define FIREQ_KV4_WS_H

#include "fireq.h"

#ifdef __cplusplus
extern "C" {
#endif

size_t fq_kv4_output_workspace_bytes(int H, int R, int T);
int fq_kv4_output_ws(const uint8_t *P_fp8, const float *p_scale, const uint8_t *V_packed,
                     const uint8_t *v_scale, uint16_t *O_bf16, int H, int R, int T, int ldp,
                     void *workspace, size_t workspace_bytes, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* FIREQ_KV4_WS_H */
