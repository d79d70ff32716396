// Host-side argument checks shared by the C-ABI sources.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "specquant.h"

namespace {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Byte ranges [a, a + na) and [b, b + nb) intersect.
inline bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  if (!a || !b || na == 0 || nb == 0) return false;
  const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
  return pa < pb + nb && pb < pa + na;
}

struct Range {
  const void* p;
  size_t n;
};

// Every output range against every input range and every other output range.
template <size_t NO, size_t NI>
bool any_alias(const Range (&outs)[NO], const Range (&ins)[NI]) {
  for (size_t i = 0; i < NO; ++i) {
    for (size_t j = 0; j < NI; ++j)
      if (overlap(outs[i].p, outs[i].n, ins[j].p, ins[j].n)) return true;
    for (size_t j = i + 1; j < NO; ++j)
      if (overlap(outs[i].p, outs[i].n, outs[j].p, outs[j].n)) return true;
  }
  return false;
}

inline sq_status device_status(hipError_t e) {
  if (e == hipSuccess) return SQ_OK;
  if (e == hipErrorStreamCaptureUnsupported) return SQ_ERR_CAPTURE;  // the workspace would have to grow
  return SQ_ERR_DEVICE;
}

// The fused projections: a kernel without the fused form returns
// hipErrorNotSupported before it enqueues anything.
inline sq_status fused_status(hipError_t e) {
  return e == hipErrorNotSupported ? SQ_ERR_UNSUPPORTED : device_status(e);
}

constexpr int64_t kMaxK = int64_t(1) << 20;
constexpr int64_t kMaxN = 0x7FFFFFFF;
constexpr int64_t kMaxHidden = 16384;

// Shared limits of the block layout of the rope / attention calls (prefill blocks: up to len_bound rows).
sq_status check_block(int32_t b, int32_t rows_per_seq, int32_t hq, int32_t hkv, int64_t len_bound,
                      int64_t capacity, int64_t rows_max = 64) {
  if (b < 1 || rows_per_seq < 1 || rows_per_seq > rows_max || hkv < 1 || hq < hkv || hq > 128 || hq % hkv != 0)
    return SQ_ERR_SHAPE;
  if (capacity < 64 || capacity > kMaxN || capacity % 64 != 0 || len_bound < 1 || len_bound > capacity)
    return SQ_ERR_SHAPE;
  if ((int64_t)b * rows_per_seq > kMaxN || (int64_t)b * hkv > 65535) return SQ_ERR_SHAPE;
  return SQ_OK;
}

}  // namespace
