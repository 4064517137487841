// The row-wise pieces of the decoder-layer prefill slice between its library
// GEMMs: RMSNorm and the SwiGLU product.
// bf16 in and out, fp32 arithmetic.
//
// All are bound by HBM: each operand is read once and each result written
// once, 16 bytes a lane.  As separate framework operations (to fp32, square,
// mean, add, rsqrt, three products, to bf16) a norm of 16,640 x 4,096 took
// 475 us and the SwiGLU product of 16,640 x 14,336 436; fused 45 and
// 227 (6.3 TB/s).

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "sift_internal.h"

namespace sift {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float lo_f(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float hi_f(uint32_t w) {
  return __builtin_bit_cast(float, w & 0xffff0000u);
}
__device__ __forceinline__ uint32_t pack(float lo, float hi) {  // round to nearest even
  const bf16x2 v = bf16x2{static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, v);
}

constexpr int kThreads = 256;

// One workgroup per row; a thread keeps kV 16-byte chunks of the row in
// registers between the sum of squares and the output (out may be x).
template <int kV>
__global__ __launch_bounds__(kThreads) void rms_norm_kernel(const u32x4* x,
                                                            const u32x4* __restrict__ weight,
                                                            int chunks, float inv_width, float eps,
                                                            u32x4* out) {
  __shared__ float part[kThreads / 64];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * chunks;
  const int t = threadIdx.x;
  u32x4 v[kV];
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < kV; ++i) {
    const int c = t + kThreads * i;
    v[i] = u32x4{0u, 0u, 0u, 0u};
    if (c < chunks) v[i] = x[base + c];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = lo_f(v[i][e]), b = hi_f(v[i][e]);
      sq = fmaf(a, a, sq);
      sq = fmaf(b, b, sq);
    }
  }
  for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
  if ((t & 63) == 0) part[t >> 6] = sq;
  __syncthreads();
  sq = (part[0] + part[1]) + (part[2] + part[3]);
  const float r = rsqrtf(sq * inv_width + eps);
#pragma unroll
  for (int i = 0; i < kV; ++i) {
    const int c = t + kThreads * i;
    if (c >= chunks) break;
    const u32x4 w = weight[c];
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = pack(lo_f(v[i][e]) * r * lo_f(w[e]), hi_f(v[i][e]) * r * hi_f(w[e]));
    out[base + c] = y;
  }
}

__device__ __forceinline__ float silu(float x) { return x / (1.f + expf(-x)); }

__global__ __launch_bounds__(kThreads) void silu_mul_kernel(const u32x4* gate, const u32x4* up,
                                                            int64_t chunks, u32x4* out) {
  const int64_t step = static_cast<int64_t>(gridDim.x) * kThreads;
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; c < chunks; c += step) {
    const u32x4 g = gate[c], u = up[c];
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = pack(silu(lo_f(g[e])) * lo_f(u[e]), silu(hi_f(g[e])) * hi_f(u[e]));
    out[c] = y;
  }
}

}  // namespace

hipError_t launch_rms_norm(const void* x, const void* weight, int64_t rows, int width, float eps,
                           void* out, hipStream_t stream) {
  if (width % 8 != 0 || width > kMaxNormWidth) return hipErrorInvalidValue;
  static_assert(kMaxNormWidth == 8 * 8 * kThreads, "eight chunks per thread");
  const int chunks = width / 8;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(rows)), dim3(kThreads), 0, stream,
                       static_cast<const u32x4*>(x), static_cast<const u32x4*>(weight), chunks,
                       1.f / static_cast<float>(width), eps, static_cast<u32x4*>(out));
  };
  if (chunks <= kThreads) go(rms_norm_kernel<1>);
  else if (chunks <= 2 * kThreads) go(rms_norm_kernel<2>);
  else if (chunks <= 4 * kThreads) go(rms_norm_kernel<4>);
  else go(rms_norm_kernel<8>);
  return hipGetLastError();
}

hipError_t launch_silu_mul(const void* gate, const void* up, int64_t count, void* out,
                           hipStream_t stream) {
  const int64_t chunks = count / 8;
  const int64_t grid = std::min<int64_t>((chunks + kThreads - 1) / kThreads, 1 << 20);
  hipLaunchKernelGGL(silu_mul_kernel, dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, stream,
                     static_cast<const u32x4*>(gate), static_cast<const u32x4*>(up), chunks,
                     static_cast<u32x4*>(out));
  return hipGetLastError();
}

}  // namespace sift
