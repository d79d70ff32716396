/*
 * specquant_prefill.h -- the passes that fill a cache from a prompt.
 *
 * The projections, the rotation with its cache write and the attention of
 * specquant.h for blocks of more than 64 rows: prompts of hundreds to
 * thousands of tokens go through a model in one pass instead of in blocks of
 * 64.  The conventions of specquant.h hold (device pointers, alignment,
 * statuses, the library workspace, one stream per device); formulas, layouts
 * and device status bits are those of the calls named below, at their
 * precision: fp32 sums of exact products of the fp16 activations with the fp16
 * weights, the INT4 codes minus zero (scaled per 128-element group in fp32) or
 * the decoded FP8 codes (scaled per row in fp32).
 */
#ifndef SPECQUANT_PREFILL_H
#define SPECQUANT_PREFILL_H

#include "specquant.h"

#ifdef __cplusplus
extern "C" {
#endif

/* What a projection does with y[m][n] = x . W'^T. */
typedef enum sq_prefill_out {
  SQ_PREFILL_STORE = 0, /* y (fp32 [m][n]) = */
  SQ_PREFILL_ADD = 1,   /* y (fp32 [m][n]) += (the residual stream) */
  SQ_PREFILL_SILU = 2   /* rows [0, n/2) of W' are gates, [n/2, n) ups: y (fp16 [m][n/2]) = silu(gate) * up */
} sq_prefill_out;

/*
 * sq_verify_gemm_f16, sq_qgemv_w4a16 and sq_qgemv_w8a16 at any number of rows:
 *   1 <= m <= 2^20, k % 64 == 0 (INT4: k % 128 == 0), n * k < 2^31,
 *   64 <= k <= 2^20 (n even with SQ_PREFILL_SILU), y 16-byte aligned.
 * SQ_ERR_UNSUPPORTED (nothing enqueued): an output form or shape without a
 * kernel (an output of more than 2^22 tiles of 128 x 256).
 * Where the output has fewer tiles than the GPU has CUs, K parts' fp32 partial
 * outputs take up to 128 MB (4 m n bytes a part) of the library workspace, which
 * is not given back.
 */
sq_status sq_prefill_linear_f16(const uint16_t* x, int64_t m, int64_t k, const uint16_t* w16, int64_t n, void* y,
                                sq_prefill_out out, hipStream_t stream);
sq_status sq_prefill_linear_w4(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const uint16_t* scales,
                               const uint16_t* zeros, int64_t n, void* y, sq_prefill_out out, hipStream_t stream);
sq_status sq_prefill_linear_w8(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const float* scales,
                               int64_t n, void* y, sq_prefill_out out, hipStream_t stream);

/* sq_rope_kv_f16 (the same bits) and sq_attention_f16 with rows_per_seq up to
 * len_bound: every argument as there. */
sq_status sq_prefill_rope_kv_f16(const float* qkv, const uint16_t* bias, int32_t b, int32_t rows_per_seq, int32_t hq,
                                 int32_t hkv, const int32_t* pos_base, int32_t pos_offset, int64_t len_bound,
                                 int64_t capacity, double theta, uint16_t* q_out, uint16_t* k_cache, uint16_t* v_cache,
                                 int32_t* status, hipStream_t stream);
sq_status sq_prefill_attention_f16(const uint16_t* q, const uint16_t* k_cache, const uint16_t* v_cache, int32_t b,
                                   int32_t rows_per_seq, int32_t hq, int32_t hkv, const int32_t* pos_base,
                                   int32_t pos_offset, int64_t len_bound, int64_t capacity, uint16_t* out,
                                   hipStream_t stream);

#ifdef __cplusplus
}
#endif

#endif /* SPECQUANT_PREFILL_H */
