// C ABI of the pieces the decoder-layer prefill slice adds around the sparse
// attention: the rotary position embedding (rope.hip), the norms and the
// SwiGLU product (layer_ops.hip).  The projections are library GEMMs called
// by the caller.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "layer_api.h"
#include "sift.h"
#include "sift_internal.h"

namespace {
bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }
}  // namespace

extern "C" {

sift_status sift_rope(const sift_tensor* q, const sift_tensor* k, const int32_t* positions,
                      const float* inv_freq, void* stream) {
  if (q == nullptr || k == nullptr) return SIFT_E_NULL;
  if (q->tokens > 0 && (q->data == nullptr || k->data == nullptr || positions == nullptr ||
                        inv_freq == nullptr))
    return SIFT_E_NULL;
  if (q->tokens != k->tokens || q->tokens < 0) return SIFT_E_SHAPE;
  if (q->head_dim != k->head_dim || q->heads < 1 || k->heads < 1) return SIFT_E_SHAPE;
  if (q->dtype != SIFT_BF16 || k->dtype != SIFT_BF16) return SIFT_E_UNSUPPORTED;
  if (q->head_dim < 2 || q->head_dim % 2 != 0) return SIFT_E_UNSUPPORTED;
  if (q->tokens == 0) return SIFT_OK;
  const hipError_t e = sift::launch_rope(q->data, q->tokens, q->heads, k->data, k->heads,
                                         q->head_dim, positions, inv_freq,
                                         static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

sift_status sift_layer_rms_norm(const void* x, const void* weight, int64_t rows, int32_t width,
                                float eps, void* out, void* stream) {
  if (rows < 0 || width < 1) return SIFT_E_SHAPE;
  if (rows == 0) return SIFT_OK;
  if (x == nullptr || weight == nullptr || out == nullptr) return SIFT_E_NULL;
  if (width % 8 != 0 || width > sift::kMaxNormWidth) return SIFT_E_UNSUPPORTED;
  if (!aligned16(x) || !aligned16(weight) || !aligned16(out)) return SIFT_E_UNSUPPORTED;
  if (rows >= int64_t(1) << 24) return SIFT_E_CAPACITY;  // a grid holds fewer than 2^32 threads
  const hipError_t e = sift::launch_rms_norm(x, weight, rows, width, eps, out,
                                             static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

sift_status sift_layer_silu_mul(const void* gate, const void* up, int64_t count, void* out,
                                void* stream) {
  if (count < 0) return SIFT_E_SHAPE;
  if (count == 0) return SIFT_OK;
  if (gate == nullptr || up == nullptr || out == nullptr) return SIFT_E_NULL;
  if (count % 8 != 0 || !aligned16(gate) || !aligned16(up) || !aligned16(out))
    return SIFT_E_UNSUPPORTED;
  const hipError_t e =
      sift::launch_silu_mul(gate, up, count, out, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

}  // extern "C"
