// C entries that the Python package's decoder layer calls: not part of the
// ABI in include/sift.h.
#pragma once

#include <stdint.h>

#include "sift.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * The row-wise pieces of the decoder-layer prefill slice between its GEMMs,
 * bf16 in and out with fp32 arithmetic, in device memory, 16-byte aligned.
 *
 * sift_layer_rms_norm: out = x / sqrt(mean(x^2) + eps) * weight for each of
 *   `rows` rows of `width` values.  out may be x.
 * sift_layer_silu_mul: out[i] = gate[i] / (1 + exp(-gate[i])) * up[i],
 *   i < count, rounded once.  out may be gate or up.
 * Errors: SIFT_E_NULL; SIFT_E_SHAPE (rows or count < 0, width < 1);
 *   SIFT_E_UNSUPPORTED (width or count not a multiple of 8, width above 16384,
 *   misaligned); SIFT_E_CAPACITY (2^24 rows or more); SIFT_E_HIP.
 */
sift_status sift_layer_rms_norm(const void* x, const void* weight, int64_t rows, int32_t width,
                                float eps, void* out, void* stream);
sift_status sift_layer_silu_mul(const void* gate, const void* up, int64_t count, void* out,
                                void* stream);

#ifdef __cplusplus
}
#endif
