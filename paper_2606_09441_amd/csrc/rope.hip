// Rotary position embedding of q and k, in place, for the decoder-layer
// prefill slice at the Llama-3.1-8B shape (the model of Section 6).  Rotate-
// half form: for i < D/2, with angle a = pos * inv_freq[i] (an fp32 product),
//   x[i]       <- x[i] cos a - x[i + D/2] sin a
//   x[i + D/2] <- x[i + D/2] cos a + x[i] sin a
// inv_freq is given by the caller, so any frequency schedule (plain base^-2i/D
// or a rescaled one) is one table.  bf16 in and out, fp32 arithmetic.

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "sift_internal.h"

namespace sift {
namespace {

__device__ __forceinline__ float bf2f(uint16_t b) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(b) << 16);
}

__device__ __forceinline__ uint16_t f2bf(float f) {  // round to nearest even
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__global__ __launch_bounds__(256) void rope_kernel(uint16_t* __restrict__ x, int64_t rows, int heads,
                                                   int half, const int32_t* __restrict__ pos,
                                                   const float* __restrict__ inv_freq) {
  const int64_t n = rows * heads * half;
  for (int64_t t = blockIdx.x * 256 + threadIdx.x; t < n; t += static_cast<int64_t>(gridDim.x) * 256) {
    const int i = static_cast<int>(t % half);
    const int64_t rh = t / half;              // token * heads + head
    const int64_t tok = rh / heads;
    const float a = static_cast<float>(pos[tok]) * inv_freq[i];
    float s, c;
    sincosf(a, &s, &c);
    uint16_t* p = x + rh * (2 * half);
    const float x1 = bf2f(p[i]), x2 = bf2f(p[i + half]);
    p[i] = f2bf(x1 * c - x2 * s);
    p[i + half] = f2bf(x2 * c + x1 * s);
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRopeTokens = 4;    // tokens of a workgroup
constexpr int kMaxHalf = 256;

// The same for halves of whole 16-byte chunks (half a multiple of 8): a
// workgroup takes four tokens, forms each (token, i) sine and cosine once, in
// LDS, and rotates every head of q and of k with them, 16 bytes of each half
// a thread.  Bound by HBM: with a sine and cosine per head and 2-byte accesses
// 16,640 tokens x 40 heads x 128 took 157 us in two launches, this 54.
__global__ __launch_bounds__(256) void rope_rows_kernel(uint16_t* __restrict__ q, int hq,
                                                        uint16_t* __restrict__ k, int hkv,
                                                        int64_t tokens, int half,
                                                        const int32_t* __restrict__ pos,
                                                        const float* __restrict__ inv_freq) {
  __shared__ float sn[kRopeTokens * kMaxHalf], cs[kRopeTokens * kMaxHalf];
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kRopeTokens;
  const int nt = static_cast<int>(min(static_cast<int64_t>(kRopeTokens), tokens - t0));
  for (int e = threadIdx.x; e < nt * half; e += 256) {
    const int t = e / half, i = e - t * half;
    sincosf(static_cast<float>(pos[t0 + t]) * inv_freq[i], &sn[e], &cs[e]);
  }
  __syncthreads();
  const int per = half / 8;       // chunks of a half
  const int heads = hq + hkv;
  for (int e = threadIdx.x; e < nt * heads * per; e += 256) {
    const int c = e % per, th = e / per;
    const int t = th / heads, h = th - t * heads;
    uint16_t* p = h < hq ? q + ((t0 + t) * hq + h) * (2 * half)
                         : k + ((t0 + t) * hkv + (h - hq)) * (2 * half);
    u32x4* lo = reinterpret_cast<u32x4*>(p + 8 * c);
    u32x4* hi = reinterpret_cast<u32x4*>(p + half + 8 * c);
    const u32x4 a = *lo, b = *hi;
    u32x4 x, y;
    const float* s = sn + t * half + 8 * c;
    const float* g = cs + t * half + 8 * c;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      uint16_t rx[2], ry[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float x1 = bf2f(static_cast<uint16_t>(a[w] >> (16 * j)));
        const float x2 = bf2f(static_cast<uint16_t>(b[w] >> (16 * j)));
        rx[j] = f2bf(x1 * g[2 * w + j] - x2 * s[2 * w + j]);
        ry[j] = f2bf(x2 * g[2 * w + j] + x1 * s[2 * w + j]);
      }
      x[w] = rx[0] | static_cast<uint32_t>(rx[1]) << 16;
      y[w] = ry[0] | static_cast<uint32_t>(ry[1]) << 16;
    }
    *lo = x;
    *hi = y;
  }
}

}  // namespace

hipError_t launch_rope(void* q, int64_t tokens, int hq, void* k, int hkv, int head_dim,
                       const int32_t* positions, const float* inv_freq, hipStream_t stream) {
  const int half = head_dim / 2;
  // rows of whole aligned chunks, q and k apart; a grid holds fewer than 2^32
  // threads
  const int64_t qn = tokens * hq * half * 2, kn = tokens * hkv * half * 2;
  uint16_t* const qx = static_cast<uint16_t*>(q);
  uint16_t* const kx = static_cast<uint16_t*>(k);
  if ((qx + qn <= kx || kx + kn <= qx) && half % 8 == 0 && half <= kMaxHalf && reinterpret_cast<uintptr_t>(q) % 16 == 0 &&
      reinterpret_cast<uintptr_t>(k) % 16 == 0 && tokens < int64_t(1) << 25) {
    const int64_t g = (tokens + kRopeTokens - 1) / kRopeTokens;
    hipLaunchKernelGGL(rope_rows_kernel, dim3(static_cast<unsigned>(g)), dim3(256), 0, stream, qx,
                       hq, kx, hkv, tokens, half, positions, inv_freq);
    return hipGetLastError();
  }
  for (int pass = 0; pass < 2; ++pass) {
    void* x = pass == 0 ? q : k;
    const int heads = pass == 0 ? hq : hkv;
    const int64_t n = tokens * heads * half;
    if (n == 0) continue;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(rope_kernel, dim3(static_cast<unsigned>(g)), dim3(256), 0, stream,
                       static_cast<uint16_t*>(x), tokens, heads, half, positions, inv_freq);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sift
