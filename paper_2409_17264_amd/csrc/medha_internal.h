/* Entry points of libmedha.so for the package's own binding. */
#ifndef MEDHA_INTERNAL_H_
#define MEDHA_INTERNAL_H_

#include "medha.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Device memory of at least `bytes` bytes, 256-byte aligned, or NULL. */
typedef void* (*medha_alloc)(size_t bytes, void* context);

/* medha_chunked_prefill_attn with a workspace of the size that the query reports, asked for once the
 * batch is planned: one plan for the size and the call. */
int medha_chunked_prefill_attn_alloc(const void* q, const medha_kv_cache* kv,
                                     const int32_t* page_table, const int64_t* page_table_offs,
                                     const int32_t* prefix_len, const int32_t* chunk_len,
                                     int32_t batch, int32_t num_q_heads, float softmax_scale,
                                     float* out, float* lse, medha_alloc alloc, void* context,
                                     void* hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* MEDHA_INTERNAL_H_ */
