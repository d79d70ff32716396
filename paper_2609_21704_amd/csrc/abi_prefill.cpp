// C ABI of the prefill passes: host-side argument validation and dispatch.
#include <math.h>

#include "abi_checks.hpp"
#include "sq_internal.hpp"
#include "specquant_prefill.h"

extern "C" {

sq_status sq_prefill_rope_kv_f16(const float* qkv, const uint16_t* bias, int32_t b, int32_t rows_per_seq, int32_t hq,
                                 int32_t hkv, const int32_t* pos_base, int32_t pos_offset, int64_t len_bound,
                                 int64_t capacity, double theta, uint16_t* q_out, uint16_t* k_cache, uint16_t* v_cache,
                                 int32_t* status, hipStream_t stream) {
  if (!qkv || !pos_base || !q_out || !k_cache || !v_cache) return SQ_ERR_NULL;
  const sq_status bs = check_block(b, rows_per_seq, hq, hkv, len_bound, capacity, len_bound);
  if (bs != SQ_OK) return bs;
  if (b > 65535) return SQ_ERR_SHAPE;
  if (!isfinite(theta)) return SQ_ERR_NONFINITE;
  if (!(theta > 1.0)) return SQ_ERR_SHAPE;
  if (!aligned(qkv, 16) || !aligned(bias, 16) || !aligned(pos_base, 4) || !aligned(q_out, 16) ||
      !aligned(k_cache, 16) || !aligned(v_cache, 16) || !aligned(status, 4))
    return SQ_ERR_ALIGN;
  const size_t m = (size_t)b * rows_per_seq, nh = (size_t)hq + 2 * (size_t)hkv;
  const size_t cache = (size_t)b * hkv * capacity * 128 * 2;
  const Range outs[] = {{q_out, m * hq * 128 * 2}, {k_cache, cache}, {v_cache, cache}, {status, 4}};
  const Range ins[] = {{qkv, m * nh * 128 * 4}, {bias, nh * 128 * 2}, {pos_base, (size_t)b * 4}};
  if (any_alias(outs, ins)) return SQ_ERR_ALIAS;
  (void)hipGetLastError();
  return device_status(sq::launch_prefill_rope_kv(qkv, bias, b, rows_per_seq, hq, hkv, pos_base, pos_offset, len_bound,
                                                  capacity, theta, q_out, k_cache, v_cache, status, stream));
}

sq_status sq_prefill_attention_f16(const uint16_t* q, const uint16_t* k_cache, const uint16_t* v_cache, int32_t b,
                                   int32_t rows_per_seq, int32_t hq, int32_t hkv, const int32_t* pos_base,
                                   int32_t pos_offset, int64_t len_bound, int64_t capacity, uint16_t* out,
                                   hipStream_t stream) {
  if (!q || !k_cache || !v_cache || !pos_base || !out) return SQ_ERR_NULL;
  const sq_status bs = check_block(b, rows_per_seq, hq, hkv, len_bound, capacity, len_bound);
  if (bs != SQ_OK) return bs;
  if (b > 65535) return SQ_ERR_SHAPE;
  if (!aligned(q, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16) || !aligned(pos_base, 4) ||
      !aligned(out, 16))
    return SQ_ERR_ALIGN;
  const size_t m = (size_t)b * rows_per_seq;
  const size_t cache = (size_t)b * hkv * capacity * 128 * 2;
  const Range outs[] = {{out, m * hq * 128 * 2}};
  const Range ins[] = {{q, m * hq * 128 * 2}, {k_cache, cache}, {v_cache, cache}, {pos_base, (size_t)b * 4}};
  if (any_alias(outs, ins)) return SQ_ERR_ALIAS;
  (void)hipGetLastError();
  return device_status(sq::launch_prefill_attention(q, k_cache, v_cache, b, rows_per_seq, hq, hkv, capacity, pos_base,
                                                    pos_offset, len_bound, out, stream));
}

}  // extern "C"

namespace {

// Validation shared by the prefill projections; wbytes, sbytes, zbytes: sizes of
// the weights and of their scales and zeros.
sq_status check_prefill(const uint16_t* x, int64_t m, int64_t k, int64_t kgrain, const Range& w, const Range& scales,
                        const Range& zeros, int64_t n, const void* y, int out) {
  if (!x || !w.p || !y) return SQ_ERR_NULL;
  if (m < 1 || m > kMaxK || n < 1 || n > kMaxN || k < kgrain || k > kMaxK || k % kgrain != 0 ||
      n * k > int64_t(0x7FFFFFFF))
    return SQ_ERR_SHAPE;
  if (out != SQ_PREFILL_STORE && out != SQ_PREFILL_ADD && out != SQ_PREFILL_SILU) return SQ_ERR_UNSUPPORTED;
  if (out == SQ_PREFILL_SILU && n % 2 != 0) return SQ_ERR_SHAPE;
  if (!aligned(x, 16) || !aligned(w.p, 16) || !aligned(y, 16)) return SQ_ERR_ALIGN;
  const Range outs[] = {{y, out == SQ_PREFILL_SILU ? (size_t)m * n : (size_t)m * n * 4}};
  const Range ins[] = {{x, (size_t)m * k * 2}, w, scales, zeros};
  return any_alias(outs, ins) ? SQ_ERR_ALIAS : SQ_OK;
}

}  // namespace

extern "C" {

sq_status sq_prefill_linear_f16(const uint16_t* x, int64_t m, int64_t k, const uint16_t* w16, int64_t n, void* y,
                                sq_prefill_out out, hipStream_t stream) {
  const sq_status st = check_prefill(x, m, k, 64, {w16, (size_t)n * k * 2}, {nullptr, 0}, {nullptr, 0}, n, y, out);
  if (st != SQ_OK) return st;
  (void)hipGetLastError();
  return fused_status(sq::launch_prefill_f16(x, m, k, w16, n, y, out, stream));
}

sq_status sq_prefill_linear_w4(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const uint16_t* scales,
                               const uint16_t* zeros, int64_t n, void* y, sq_prefill_out out, hipStream_t stream) {
  if (!scales || !zeros) return SQ_ERR_NULL;
  if (!aligned(scales, 2) || !aligned(zeros, 2)) return SQ_ERR_ALIGN;
  const size_t nk = (size_t)n * (size_t)k;
  const sq_status st = check_prefill(x, m, k, 128, {codes, nk / 2}, {scales, nk / 64}, {zeros, nk / 64}, n, y, out);
  if (st != SQ_OK) return st;
  (void)hipGetLastError();
  return fused_status(sq::launch_prefill_w4(x, m, k, codes, scales, zeros, n, y, out, stream));
}

sq_status sq_prefill_linear_w8(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const float* scales,
                               int64_t n, void* y, sq_prefill_out out, hipStream_t stream) {
  if (!scales) return SQ_ERR_NULL;
  if (!aligned(scales, 4)) return SQ_ERR_ALIGN;
  const sq_status st =
      check_prefill(x, m, k, 64, {codes, (size_t)n * k}, {scales, (size_t)n * 4}, {nullptr, 0}, n, y, out);
  if (st != SQ_OK) return st;
  (void)hipGetLastError();
  return fused_status(sq::launch_prefill_w8(x, m, k, codes, scales, n, y, out, stream));
}

}  // extern "C"
