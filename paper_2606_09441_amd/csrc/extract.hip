// Offline metadata extraction on the GPU (Sections 4.1, 4.2; the metadata is
// made by a dense standalone prefill of each document, Section 4.4).
//
// For every document, query head and block of 128 query rows, one workgroup
// (4 wavefronts x 32 rows) walks the causal key blocks of 64 keys:
//
//   pass 1: S^T = K Q^T on v_mfma_f32_32x32x16_bf16 (queries on lanes, as in
//           the attention kernel), running row max m and row sum l of
//           exp2(c S - m), c = scale * log2(e); each row's largest S of every
//           tile of the block stays in LDS;
//   pass 2: probability A = exp2(c S - m) / l exceeds a threshold t exactly
//           when S > (log2 t + log2 l + m) / c, so the decisions need no
//           exponential.  LA: a tile's flag is set when any of its cells
//           passes alpha, that is when one of its row maxima does: no scores
//           are formed again.  CA: the cells of each key page that pass beta
//           are counted (ballot popcounts, one atomic add per page and
//           wavefront), from the scores formed again, but only of blocks
//           where some row maximum passes beta.
//
// Bound by VALU issue in pass 1: an FMA, an exponential, an add and half a max
// per score beside the 16 MFMAs of a block.  By the counters the matrix cores
// are busy 44% of the SIMD cycles, a block takes 33 exponentials, 10.3 vector
// instructions are issued per MFMA (pass 2 included), and wavefronts wait to
// issue for 41% of their time: so what counts is fewer of them and more
// wavefronts to fill waits: one K block in LDS and 110 registers give four on a
// SIMD.  32 documents x
// 2048 tokens x 48 heads (T = 64, D = 128): 2.17 ms with all scores formed
// twice and two compares each in pass 2; with the row maxima 1.53 ms at three
// wavefronts, 1.19 at four; exponentials interleaved by hand with the next
// block's MFMAs (184 registers, two or three wavefronts) 1.72 and 1.43.  With
// every block passing beta it is 1.78 ms (2.21 before).
// Key blocks beyond those whose maxima fit LDS (kMaxBytes) take both
// decisions from scores formed again.
//
// A pack pass then turns flags into LA bits and counts into CA bits (count >
// gamma * the page's causal cells), MSB first, document-major with the query
// heads inside each document: the layout the online path reads.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "sift_internal.h"

namespace sift {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kQB = 128;  // query rows per workgroup
constexpr int kKB = 64;   // keys per block
// LDS for the row maxima.  Beside the 64 D bf16 of the K block this keeps
// three (D = 128) or four to five workgroups (D = 64) on a CU for documents
// of any length; more of it costs residency, less of it more blocks whose
// scores are formed again.  us at 24 / 32 / 48 KB (16 documents x 2048, 32/8
// heads, then 2 x 12000): T = 64, D = 128 446 / 446 / 446, 2403 / 2170 / 2256;
// T = 64, D = 64 324 / 323 / 323, 1624 / 1704 / 1931; T = 16, D = 128
// 627 / 594 / 684, 3007 / 2997 / 3474; T = 16, D = 64 486 / 525 / 612,
// 2285 / 2530 / 3151.
template <int D>
constexpr int kMaxBytes = D == 64 ? 24 << 10 : 32 << 10;

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Key index (inside the 64-key block) of accumulator a, register j of a lane
// in half hf of the wavefront (32x32 MFMA output layout).
__device__ __forceinline__ int key_of(int a, int j, int hf) {
  return 32 * a + 8 * (j >> 2) + 4 * hf + (j & 3);
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4u __attribute__((ext_vector_type(4), aligned(2)));  // off a 16-byte line
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) __bf16 lds_bf16;
constexpr int kBufferWord3 = 0x00020000;  // gfx9-family raw buffer resource word 3

// Global -> LDS, 16 bytes per lane from byte voff of the resource, landing
// at m0 + 16 * lane.
__device__ __forceinline__ void dma_b128(int m0, int voff, const i32x4& rs) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(m0), "v"(voff), "s"(rs)
               : "memory", "m0");
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The larger of x in lane l and lane l ^ 32 (inline asm: the builtin's two
// results are folded into one when both inputs are the same value).
__device__ __forceinline__ float swap_max(float x) {
  float u = x, v = x;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(u), "+v"(v));
  return fmaxf(u, v);
}

// S^T for 64 keys x this wavefront's 32 queries: s[0] keys 0..31, s[1] 32..63.
// Lane (l32, hf) reads row 32 a + l32, chunk 2 k + hf, stored at chunk
// (2 k + hf) ^ (row & (chunks - 1)): its address for k = 0 XORed with 32 k.
// The fragments of two k-steps are in flight, held to that order by the
// scheduling barriers.
template <int D>
__device__ __forceinline__ void scores(const __bf16* lds, const bf16x8 (&qf)[D / 16], int l32, int hf,
                                       f32x16 (&s)[2]) {
  constexpr int kCpr = D / 8, kN = D / 16, kAhead = 2;
  const int base = (l32 * kCpr + (hf ^ (l32 & (kCpr - 1)))) * 16;  // bytes
  const char* p = reinterpret_cast<const char*>(lds);
  bf16x8 f[kAhead][2];
  auto frag = [&](int k, int a) {
    return *reinterpret_cast<const bf16x8*>(p + ((base ^ (k << 5)) + a * 32 * D * 2));
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k)
#pragma unroll
    for (int a = 0; a < 2; ++a) f[k][a] = frag(k, a);
#pragma unroll
  for (int k = 0; k < kN; ++k) {
#pragma unroll
    for (int a = 0; a < 2; ++a) s[a] = mfma(f[k % kAhead][a], qf[k], k == 0 ? f32x16{} : s[a]);
    if (k + kAhead < kN) {
#pragma unroll
      for (int a = 0; a < 2; ++a) f[k % kAhead][a] = frag(k + kAhead, a);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// kDma: K starts on a 16-byte line and is staged by DMA; else through registers.
template <int D, int T, bool kDma>
__global__ __launch_bounds__(256, 4) void extract_kernel(ExtractArgs a, int cap) {
  constexpr int kKS = D / 16;
  constexpr int kSub = T < kKB ? kKB / T : 1;  // tiles of a key block
  constexpr int kCpr = D / 8;                  // 16-byte chunks of a key row
  constexpr int kDmaRows = 64 / kCpr;          // key rows of one DMA instruction
  // one K block, refilled while its scores are used.  16-byte chunks, chunk
  // index XOR (row & (chunks per row - 1)), so that the 32 rows read by one
  // MFMA fragment spread over the banks
  __shared__ __attribute__((aligned(1024))) __bf16 lds[kKB * D];
  // blocks kb < cap: each row's largest score per tile, [cap][kSub][kQB], and
  // the wavefronts that have to count in the block
  extern __shared__ float rowmax[];
  __shared__ int need[kMaxBytes<D> / (kQB * 4)];

  const int2 bl = a.blocks[blockIdx.x];  // {document, query block}, longest first
  const ExtractDoc dc = a.docs[bl.x];
  const int h = blockIdx.y;
  const int kvh = h / (a.hq / a.hkv);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  const int row0 = bl.y * kQB + wave * 32;  // first query row of this wavefront
  const int p = row0 + l32;                 // this lane's query row (in the document)
  const int L = dc.len;

  bf16x8 qf[kKS];
  {
    const __bf16* src = a.q + (static_cast<int64_t>(dc.tok0 + p) * a.hq + h) * D + 8 * hf;
#pragma unroll
    for (int k = 0; k < kKS; ++k) {
      u32x4 x = u32x4{0u, 0u, 0u, 0u};
      if (p < L) x = *reinterpret_cast<const u32x4u*>(src + 16 * k);
      qf[k] = __builtin_bit_cast(bf16x8, x);
    }
  }
  const int last = min(bl.y * kQB + kQB, L) - 1;  // last query row of the block
  const int nkb = last / kKB + 1;                 // causal key blocks
  const int wave_last = min(row0 + 31, L - 1);    // this wavefront's last row (may be < row0)
  const int row_bytes = a.hkv * D * 2;
  const __bf16* kdoc = a.k + static_cast<int64_t>(dc.tok0) * a.hkv * D + static_cast<int64_t>(kvh) * D;
  const float c = a.c;

  // this wavefront's quarter of a key block to LDS: rows 16 w .. + 15, those
  // past the document's end as zeros
  const int drow = lane / kCpr;
  const int off0 = (16 * wave + drow) * row_bytes +
                   (((lane % kCpr) ^ (drow & (kCpr - 1))) << 4);
  const int lds_dma = static_cast<int>(reinterpret_cast<size_t>((lds_bf16*)lds)) +
                      16 * wave * D * 2;
  auto dma = [&](int kb) {
    if constexpr (!kDma) {
      const char* src = reinterpret_cast<const char*>(kdoc) + static_cast<int64_t>(kb) * kKB * row_bytes;
#pragma unroll
      for (int it = 0; it < 16 / kDmaRows; ++it) {
        const int row = 16 * wave + it * kDmaRows + drow;
        const int off = (off0 ^ (((it * kDmaRows) & (kCpr - 1)) << 4)) + it * kDmaRows * row_bytes;
        u32x4 x = u32x4{0u, 0u, 0u, 0u};
        if (kb * kKB + row < L) x = *reinterpret_cast<const u32x4u*>(src + off);
        *reinterpret_cast<lds_u32x4*>(static_cast<size_t>(lds_dma + it * 1024 + lane * 16)) = x;
      }
      return;
    }
    const unsigned long long ad = reinterpret_cast<unsigned long long>(kdoc) +
                                  static_cast<unsigned long long>(kb) * kKB * row_bytes;
    i32x4 rs = i32x4{static_cast<int>(static_cast<unsigned>(ad)),
                     static_cast<int>((ad >> 32) & 0xffff),
                     (min(kKB, L - kb * kKB) - 1) * row_bytes + D * 2, kBufferWord3};
#pragma unroll
    for (int j = 0; j < 4; ++j) rs[j] = __builtin_amdgcn_readfirstlane(rs[j]);
#pragma unroll
    for (int it = 0; it < 16 / kDmaRows; ++it)
      dma_b128(lds_dma + it * 1024,
               (off0 ^ (((it * kDmaRows) & (kCpr - 1)) << 4)) + it * kDmaRows * row_bytes, rs);
  };

  // Cells outside the causal triangle or the document become -inf (their
  // exponential is 0 and they pass no threshold).  A block is full for a
  // wavefront when all its keys precede the wavefront's first row and all
  // its rows are in the document: then nothing is masked.
  auto mask = [&](f32x16 (&s)[2], int kb) {
    const int lim = (p < L ? p : -1) - kb * kKB - 4 * hf;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 16; ++j) s[t][j] = key_of(t, j, 0) <= lim ? s[t][j] : -INFINITY;
  };
  auto full = [&](int kb) { return kb * kKB + kKB - 1 <= row0 && row0 + 31 < L; };

  // ---- pass 1: row max m and row sum l (log2 domain; l: this lane's share).
  float m = -INFINITY, mb = 0.f, l = 0.f;
  float* const rm = rowmax + wave * 32 + l32;  // tile q of block kb: rm[(kb kSub + q) kQB]
  for (int kb = threadIdx.x; kb < cap; kb += 256) need[kb] = 0;
  // masks block kb's scores, keeps their row maxima and moves m; returns the
  // factor that moves l
  auto take = [&](f32x16 (&s)[2], int kb) {
    if (!full(kb)) mask(s, kb);
    // accumulator t, register j: key quarter 2 t + j / 8
    float mq[kSub];
#pragma unroll
    for (int q = 0; q < kSub; ++q) mq[q] = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int q = (2 * t + (j >> 3)) * kSub / 4;
        mq[q] = fmaxf(mq[q], s[t][j]);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < kSub; ++q) {
      mq[q] = swap_max(mq[q]);
      mx = fmaxf(mx, mq[q]);
      if (kb < cap && hf == 0) rm[(kb * kSub + q) * kQB] = mq[q];
    }
    const float mn = fmaxf(m, mx * c);
    // mn == -inf: no key yet (lanes past the document's end)
    mb = mn == -INFINITY ? 0.f : mn;
    const float moved = __builtin_amdgcn_exp2f(m - mb);
    m = mn;
    return moved;
  };
  dma(0);
  for (int kb = 0; kb < nkb; ++kb) {
    const bool mine = kb * kKB <= wave_last;  // else no causal cell for this wavefront
    wait_dma();
    __syncthreads();
    f32x16 s[2];
    if (mine) scores<D>(lds, qf, l32, hf, s);
    __syncthreads();
    if (kb + 1 < nkb) dma(kb + 1);
    if (mine) {
      const float moved = take(s, kb);
      // the block's exponentials are summed apart, then added to l once: added to
      // l one by one each sum is rounded at l's size, an error that grows with the
      // document (16,384 keys, all but one of equal weight: 7e-5 of l, this way
      // 3e-6).  It costs a call 0.3% (1.166 / 1.170 ms), with two or four sums too
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < 32; ++j)
        sum += __builtin_amdgcn_exp2f(fmaf(s[j >> 4][j & 15], c, -mb));
      l = fmaf(l, moved, sum);
    }
  }
  l += __shfl_xor(l, 32, 64);

  // ---- pass 2: decisions.  A > t  <=>  S > (log2 t + log2 l + m) / c
  const float ll = l > 0.f ? log2f(l) : 0.f;
  const float thr_a = (a.log2_alpha + ll + m) / c;
  const float thr_b = (a.log2_beta + ll + m) / c;
  const int nt = dc.P * (dc.P + 1) / 2;
  uint8_t* flags = a.flags + dc.flag_off + static_cast<int64_t>(h) * nt;
  int32_t* counts = a.counts + dc.cnt_off + static_cast<int64_t>(h) * dc.P;
  // f[q]: the rows (bit l32) with a cell of key quarter q above alpha
  auto set_flags = [&](int kb, const uint32_t (&f)[4]) {
    if (lane != 0) return;
    if constexpr (T == 16) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int ti = row0 / 16 + r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int tj = kb * 4 + q;
          if (((f[q] >> (16 * r)) & 0xffffu) && tj <= ti) flags[ti * (ti + 1) / 2 + tj] = 1;
        }
      }
    } else if constexpr (T == 32) {
      const int ti = row0 / 32;
      for (int q = 0; q < 2; ++q) {
        const int tj = kb * 2 + q;
        if ((f[2 * q] | f[2 * q + 1]) && tj <= ti) flags[ti * (ti + 1) / 2 + tj] = 1;
      }
    } else if constexpr (T == 64) {
      const int ti = row0 / 64;
      if ((f[0] | f[1] | f[2] | f[3]) && kb <= ti) flags[ti * (ti + 1) / 2 + kb] = 1;
    } else {  // T = 128: the tile spans the workgroup's rows and two key blocks
      const int ti = row0 / 128, tj = kb / 2;
      if ((f[0] | f[1] | f[2] | f[3]) && tj <= ti) flags[ti * (ti + 1) / 2 + tj] = 1;
    }
  };
  // ---- flags from the row maxima
  const int stored = min(nkb, cap);
  for (int kb = 0; kb < stored; ++kb) {
    if (kb * kKB > wave_last) break;
    uint32_t f[4] = {0u, 0u, 0u, 0u};
    unsigned long long above = 0ull;
#pragma unroll
    for (int q = 0; q < kSub; ++q) {
      const float v = rm[(kb * kSub + q) * kQB];
      f[q * 4 / kSub] = static_cast<uint32_t>(__ballot(v > thr_a));
      above |= __ballot(v > thr_b);
    }
    set_flags(kb, f);
    if (above != 0ull && lane == 0) atomicOr(&need[kb], 1 << wave);
  }
  __syncthreads();
  // ---- scores again: blocks with a row maximum above beta, and those >= cap
  auto next = [&](int kb) {
    while (kb < stored && __builtin_amdgcn_readfirstlane(need[kb]) == 0) ++kb;
    return kb;
  };
  int kb = next(0);
  if (kb < nkb) dma(kb);
  while (kb < nkb) {
    const int nx = next(kb + 1);
    const bool mine = kb < stored ? (__builtin_amdgcn_readfirstlane(need[kb]) >> wave) & 1
                                  : kb * kKB <= wave_last;
    wait_dma();
    __syncthreads();
    f32x16 s[2];
    if (mine) scores<D>(lds, qf, l32, hf, s);
    __syncthreads();
    if (nx < nkb) dma(nx);
    if (mine) {
      if (!full(kb)) mask(s, kb);
      // per page, the cells above beta (both halves of the wavefront hold
      // keys of the same page)
      int cnt[4] = {0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          cnt[T == 16 ? 2 * t + (j >> 3) : (T == 32 ? t : 0)] += __popcll(__ballot(s[t][j] > thr_b));
      if (kb >= stored) {
        // the lanes with a cell above alpha (a ballot per register, OR-ed per
        // quarter), the two halves folded onto 32 queries
        unsigned long long qa[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int j = 0; j < 16; ++j) qa[2 * t + (j >> 3)] |= __ballot(s[t][j] > thr_a);
        uint32_t f[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          f[q] = static_cast<uint32_t>(qa[q]) | static_cast<uint32_t>(qa[q] >> 32);
        set_flags(kb, f);
      }
      if (lane == 0) {
        if constexpr (T <= kKB) {
          constexpr int kPages = kKB / T;
#pragma unroll
          for (int q = 0; q < kPages; ++q)
            if (cnt[q] > 0) atomicAdd(&counts[kb * kPages + q], cnt[q]);
        } else {
          if (cnt[0] > 0) atomicAdd(&counts[kb / 2], cnt[0]);
        }
      }
    }
    kb = nx;
  }
}

// One workgroup per (document, head): flags -> LA bytes, counts -> CA bytes.
__global__ __launch_bounds__(256) void extract_pack(ExtractArgs a, uint8_t* __restrict__ la,
                                                    uint8_t* __restrict__ ca, int tile) {
  const ExtractDoc dc = a.docs[blockIdx.x];
  const int h = blockIdx.y;
  const int P = dc.P, L = dc.len;
  const int nt = P * (P + 1) / 2;
  const int la_n = (nt + 7) / 8, ca_n = (P + 7) / 8;
  const uint8_t* flags = a.flags + dc.flag_off + static_cast<int64_t>(h) * nt;
  const int32_t* counts = a.counts + dc.cnt_off + static_cast<int64_t>(h) * P;
  uint8_t* la_v = la + dc.la_off + static_cast<int64_t>(h) * la_n;
  uint8_t* ca_v = ca + dc.ca_off + static_cast<int64_t>(h) * ca_n;
  for (int b = threadIdx.x; b < la_n; b += 256) {
    unsigned v = 0;
    for (int i = 0; i < 8; ++i) {
      const int idx = 8 * b + i;
      if (idx < nt && flags[idx]) v |= 0x80u >> i;
    }
    la_v[b] = static_cast<uint8_t>(v);
  }
  for (int b = threadIdx.x; b < ca_n; b += 256) {
    unsigned v = 0;
    for (int i = 0; i < 8; ++i) {
      const int j = 8 * b + i;
      if (j >= P) break;
      // causal cells of page j: sum over its keys k of (L - k)
      const int64_t k0 = static_cast<int64_t>(j) * tile;
      const int64_t k1 = min(static_cast<int64_t>(L), k0 + tile);
      const int64_t n = k1 - k0;
      const int64_t cells = n * L - (k0 + k1 - 1) * n / 2;
      if (static_cast<double>(counts[j]) > a.gamma * static_cast<double>(cells)) v |= 0x80u >> i;
    }
    ca_v[b] = static_cast<uint8_t>(v);
  }
}

__global__ __launch_bounds__(256) void zero_words(uint32_t* __restrict__ p, int64_t n) {
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256)
    p[i] = 0u;
}

template <int D, int T>
void launch_extract_dt(const ExtractArgs& a, int nblocks, int max_len, hipStream_t stream) {
  constexpr int kBlockBytes = (T < kKB ? kKB / T : 1) * kQB * 4;  // a key block's row maxima
  const int cap = std::min((max_len + kKB - 1) / kKB, kMaxBytes<D> / kBlockBytes);
  if (reinterpret_cast<uintptr_t>(a.k) % 16 == 0)
    hipLaunchKernelGGL((extract_kernel<D, T, true>), dim3(nblocks, a.hq), dim3(256),
                       cap * kBlockBytes, stream, a, cap);
  else
    hipLaunchKernelGGL((extract_kernel<D, T, false>), dim3(nblocks, a.hq), dim3(256),
                       cap * kBlockBytes, stream, a, cap);
}

}  // namespace

hipError_t launch_extract(const ExtractArgs& a, int32_t num_docs, int32_t num_blocks,
                          int32_t max_len, int32_t head_dim, int32_t tile, uint32_t* zero_base, int64_t zero_words_n,
                          uint8_t* la, uint8_t* ca, hipStream_t stream) {
  if (zero_words_n > 0) {
    const int64_t g = std::min<int64_t>((zero_words_n + 255) / 256, 4096);
    hipLaunchKernelGGL(zero_words, dim3(static_cast<unsigned>(g)), dim3(256), 0, stream, zero_base,
                       zero_words_n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (num_blocks > 0) {
    if (head_dim == 128) {
      if (tile == 16) launch_extract_dt<128, 16>(a, num_blocks, max_len, stream);
      else if (tile == 32) launch_extract_dt<128, 32>(a, num_blocks, max_len, stream);
      else if (tile == 64) launch_extract_dt<128, 64>(a, num_blocks, max_len, stream);
      else launch_extract_dt<128, 128>(a, num_blocks, max_len, stream);
    } else {
      if (tile == 16) launch_extract_dt<64, 16>(a, num_blocks, max_len, stream);
      else if (tile == 32) launch_extract_dt<64, 32>(a, num_blocks, max_len, stream);
      else if (tile == 64) launch_extract_dt<64, 64>(a, num_blocks, max_len, stream);
      else launch_extract_dt<64, 128>(a, num_blocks, max_len, stream);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (num_docs > 0)
    hipLaunchKernelGGL(extract_pack, dim3(num_docs, a.hq), dim3(256), 0, stream, a, la, ca, tile);
  return hipGetLastError();
}

}  // namespace sift
