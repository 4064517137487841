// Sparse attention over decoded tile lists, fp32 inputs (SIFT, Section 5.2),
// on the fp32 matrix instruction v_mfma_f32_16x16x4_f32: T = 16, 32 or 64,
// D = 64 or 128, arithmetic in fp32 throughout.
//
// What bounds it: the matrix cores.  fp32 MFMA runs at 1/16 of the bf16 rate
// (256 flop per clock and CU): 16 keys x 16 queries take D / 2 MFMAs of 32
// clocks, so the softmax (4 scores per lane) is small beside them.
//
// In both kernels a wavefront owns 16 query rows of one M-block and takes 16
// keys at a time:
//  * S^T = K Q^T: keys on the M side.  Lane (g = l / 16, i = l % 16) supplies
//    K[key i] and Q[query i], dims 16 c + 4 g + e in MFMA (c, e): one 16-byte
//    load per c, any order of the dims being as good as another.
//  * The result has query i on lane i and key 4 g + v in register v, which is
//    the B operand of O^T += V^T P^T when step s takes keys 4 g + s: register
//    s as it is.  Its A operand is V[key 4 g + s][dim 64 c + 4 i + e] for
//    output block (c, e): one 16-byte load per (s, c).
//  * O^T then holds dims 64 c + 16 g + 4 v + e of query i: 16-byte stores.
// Rows of one M-block only ever meet the tiles it lists.
//
// attn_f32_unit_kernel runs the work units of the plan over the merged steps
// of the last decode; attn_f32_kernel reads row_ptr / col_idx (caller-given
// lists) and splits small calls finer.  At 8 x 512 + 128 tokens, 32/8 heads,
// D = 128, T = 64 (44 GF) a whole decode and attention takes 0.41 ms (108
// TFLOP/s; a large fp32 library product reaches 154 here), over caller lists
// 1.6 ms; one row at a time on the vector ALUs it took 9.1 ms.

#include "sift_internal.h"

namespace sift {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // off a 16-byte line

constexpr int kRows = 16;    // query rows of a wavefront, keys of a block
constexpr int kWaves = 4;    // wavefronts of a workgroup, 16-row blocks of a group

// Which 16-row blocks get a workgroup of their own.
enum Split : int {
  kSplitNone = 0,   // none (a launch that could not hold the extra workgroups)
  kSplitQuery = 1,  // those of groups of query rows alone
  kSplitAll = 2,    // all: fewer than kFewGroups groups
};

// Calls of fewer 64-row groups (over all heads) than this split every block
// and walk the lists; larger ones run the work units, where there are steps.
// A work unit is two groups: below 512 the units leave CUs idle and the
// longest unit (32 steps and more, some 120 us) sets the time; at 512 the
// lists' workgroups, one per block, fill the chip twice over.  The attention
// alone in us, lists / units, D = 128, T = 64 (T = 16), of documents + query:
//    64 groups (1 x 400 + 64)     20 / 47 (20 / 46)
//   264        (8 x 256 + 64)     77 / 107 (76 / 163)
//   388        (12 x 500 + 64)   208 / 240 (206 / 217), the closest of 20 layouts below 512
//   448        (2 x 1500 + 500)  134 / 261 (130 / 353)
//   488        (6 x 600 + 64)    136 / 177 (131 / 186)
// and from 512 groups on, the lists splitting query rows alone:
//   528        (8 x 256 + 64)    216 / 155 (192 / 186)
//   592        (8 x 256 + 300)   259 / 301 (235 / 310), the units' one loss of 13 layouts
//   736        (3 x 900 + 64)    312 / 208 (383 / 217)
//  1312        (20 x 500 + 200) 2069 / 603 (1825 / 555)
constexpr int kFewGroups = 512;

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 load4(const float* p) {
  return *reinterpret_cast<const f32x4u*>(p);
}
__device__ __forceinline__ void store4(float* p, f32x4 x) { *reinterpret_cast<f32x4u*>(p) = x; }

// Over the four lanes of a query (l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ __forceinline__ float quad_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

// The running row max (log2 domain) moves to the new scores' max mx where
// that is larger: O, l and the sum `part` not yet added to l are rescaled.
//
// A tile's or step's weights are summed apart, then added to l once: added to l
// one by one each sum is rounded at l's size, an error that grows with the list
// (16,384 keys, all but one of equal weight: 5e-5 of l, this way 4e-6).
template <int D>
__device__ __forceinline__ void rescale(float mx, float& mref, float& lsum, float& part,
                                        f32x4 (&o)[D / 16]) {
  if (!__builtin_amdgcn_ballot_w64(mx > mref)) return;
  const float mnew = fmaxf(mref, mx);
  const float alpha = mref == -INFINITY ? 0.f : exp2f(mref - mnew);  // O and l are 0 then
  mref = mnew;
  lsum *= alpha;
  part *= alpha;
#pragma unroll
  for (int d = 0; d < D / 16; ++d) o[d] *= alpha;
}

// ---- over lists ------------------------------------------------------------
//
// Operands come straight from memory (L1 / L2) into registers, without LDS or
// barriers: 16 KB of K and V per 16 x 16 cells at D = 128, so a large call is
// bound by the L2 (about 25 TFLOP/s).
//
// Split of the work: a group is four 16-row blocks (64 rows at T = 64).  Its
// four wavefronts normally take a block each and read the same tiles (their
// lists are the same at T = 64, nearly so below).  The rows of a user query
// list every tile of their prompt, several times a document row's list, and
// would end last: there, and in calls with too few groups to fill the chip,
// each block gets a workgroup of its own, whose wavefronts take every fourth
// tile of the list and merge their sums in LDS.  Groups run last M-block
// first (the longest lists of a prompt), and the query heads of a kv head on
// one XCD.

template <int T, int D>
__global__ __launch_bounds__(256, 4) void attn_f32_kernel(PlanTables pt, AttnArgs a, int groups,
                                                          int mode) {
  constexpr int kBlocks = T / kRows;             // 16-row blocks of a tile
  constexpr int kTiles = kWaves / kBlocks;       // tiles of a group
  constexpr int kC = D / 16;                     // 16-byte loads of a K or Q row per lane
  constexpr int kVc = D / 64;                    // 16-byte loads of a V row per lane
  constexpr int kLds = D + 4;                    // padded row of a partial result
  __shared__ __attribute__((aligned(16))) float part[kWaves][kRows * kLds];
  __shared__ float part_m[kWaves][kRows], part_l[kWaves][kRows];

  // workgroup -> (head, group, sub): XCD x (workgroups go round-robin) takes
  // the heads x hq / 8 .. when they divide, last group first
  const int subs = mode == kSplitNone ? 1 : kWaves;
  const int x = blockIdx.x % kNumXcd;
  const int sub = blockIdx.x / kNumXcd % subs;
  const int idx = blockIdx.x / (kNumXcd * subs);
  int h, grp;
  if (a.hq % kNumXcd == 0) {
    const int hc = a.hq / kNumXcd;
    h = x * hc + idx % hc;
    grp = groups - 1 - idx / hc;
  } else {
    const int r = idx * kNumXcd + x;
    h = r % a.hq;
    grp = groups - 1 - r / a.hq;
  }
  if (grp < 0) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M = pt.num_tiles;
  bool split = mode != kSplitNone;  // one block per workgroup
  if (mode == kSplitQuery) {
    for (int t = 0; t < kTiles; ++t) {
      const int mt = grp * kTiles + t;
      if (mt < M && pt.seg_kind[pt.tile_seg[mt]] != kQuery) split = false;
    }
  }
  if (!split && sub != 0) return;
  const int blk = split ? sub : wave;            // block of the group
  const int m = grp * kTiles + blk / kBlocks;
  const int bi = blk % kBlocks;                  // block of the M-block
  const int qlen = m < M ? pt.tile_len[m] - kRows * bi : 0;
  if (qlen <= 0) return;  // split: the whole workgroup; else no barrier follows

  const int lane = threadIdx.x & 63;
  const int i = lane & 15;
  const int g = lane >> 4;
  const int kvh = h / (a.hq / a.hkv);
  const float c2 = a.scale_log2;
  const int64_t qtok = static_cast<int64_t>(pt.tile_tok0[m]) + kRows * bi;

  f32x4 qf[kC];
  {
    const float* q = static_cast<const float*>(a.q) +
                     ((qtok + min(i, qlen - 1)) * a.hq + h) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < kC; ++c) qf[c] = load4(q + 16 * c);
  }
  f32x4 o[4 * kVc];
#pragma unroll
  for (int d = 0; d < 4 * kVc; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mref = -INFINITY;  // running row max, log2 domain
  float lsum = 0.f;        // this lane's share of the row sum

  const int stride = a.hkv * D;
  const float* kp = static_cast<const float*>(a.k) + kvh * D + 4 * g;
  const float* vp = static_cast<const float*>(a.v) + kvh * D + 4 * i;
  const int lo = pt.tile_lo[m];
  const int64_t row = static_cast<int64_t>(h) * M + m;
  const int64_t cap = a.col_capacity;
  const int64_t beg = min(cap, max(static_cast<int64_t>(0), static_cast<int64_t>(a.row_ptr[row])));
  const int64_t end = min(cap, max(beg, static_cast<int64_t>(a.row_ptr[row + 1])));
  for (int64_t e = beg + (split ? wave : 0); e < end; e += split ? kWaves : 1) {
    const int n = a.col_idx[e];
    if (n < lo || n > m) continue;  // outside the prompt or after the M-block
    const int64_t tok = kv_row0(pt, a.pages, n);
    const int klen = pt.tile_len[n];
    const bool diag = n == m;
    float sum = 0.f;  // the tile's weights
    for (int kb = 0; kb < kBlocks; ++kb) {
      // keys after the length or, on the diagonal, after the last query
      if (kRows * kb >= klen || (diag && kb > bi)) break;
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
      f32x4 kf[kC];
      const float* k = kp + (tok + min(kRows * kb + i, klen - 1)) * stride;
#pragma unroll
      for (int c = 0; c < kC; ++c) kf[c] = load4(k + 16 * c);
      // all of a phase's loads before its MFMAs: left to itself the compiler
      // issues and awaits two at a time, to save registers
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < kC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) s = mfma(kf[c][r], qf[c][r], s);
      f32x4 vf[4][kVc];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* v = vp + (tok + min(kRows * kb + 4 * g + r, klen - 1)) * stride;
#pragma unroll
        for (int c = 0; c < kVc; ++c) vf[r][c] = load4(v + 64 * c);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (diag || kRows * kb + kRows > klen) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = kRows * kb + 4 * g + r;
          if (key >= klen || (diag && key > kRows * bi + i)) s[r] = -INFINITY;
        }
      }
      const float mx = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * c2;
      rescale<D>(mx, mref, lsum, sum, o);
      const float base = mref == -INFINITY ? 0.f : mref;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = exp2f(fmaf(s[r], c2, -base));
        sum += p;
#pragma unroll
        for (int c = 0; c < kVc; ++c)
#pragma unroll
          for (int d = 0; d < 4; ++d) o[4 * c + d] = mfma(vf[r][c][d], p, o[4 * c + d]);
      }
    }
    lsum += sum;
  }

  lsum = quad_sum(lsum);
  float* out = static_cast<float*>(a.out);
  if (!split) {
    if (i >= qlen) return;
    const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
    float* dst = out + ((qtok + i) * a.hq + h) * D + 16 * g;
#pragma unroll
    for (int c = 0; c < kVc; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        store4(dst + 64 * c + 4 * r,
               f32x4{o[4 * c][r], o[4 * c + 1][r], o[4 * c + 2][r], o[4 * c + 3][r]} * inv);
    return;
  }
  // the wavefronts' partial sums, each relative to 2^m
#pragma unroll
  for (int c = 0; c < kVc; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f32x4*>(&part[wave][i * kLds + 64 * c + 16 * g + 4 * r]) =
          f32x4{o[4 * c][r], o[4 * c + 1][r], o[4 * c + 2][r], o[4 * c + 3][r]};
  if (g == 0) {
    part_m[wave][i] = mref;
    part_l[wave][i] = lsum;
  }
  __syncthreads();
  const int r = threadIdx.x / 16;  // query row
  if (r >= qlen) return;
  float mx = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, part_m[w][r]);
  float wt[kWaves], l = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    // a wavefront that saw no key has O = l = 0
    wt[w] = part_m[w][r] == -INFINITY ? 1.f : exp2f(part_m[w][r] - mx);
    l += part_l[w][r] * wt[w];
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
  for (int c = 0; c < kVc; ++c) {
    const int d = 64 * c + 4 * (threadIdx.x % 16);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) acc += load4(&part[w][r * kLds + d]) * wt[w];
    store4(out + ((qtok + r) * a.hq + h) * D + d, acc * inv);
  }
}

// ---- the unit kernel ------------------------------------------------------
//
// One workgroup runs one work unit of the plan (sift_internal.h): 128 query
// rows of a head (two 64-row blocks), eight wavefronts of 16 rows, over the
// merged steps that the decode wrote, in the launch order it made; long
// query units come in pieces, merged by combine_kernel.  A step is 64 keys:
// K and V go through LDS (DMA, 16-byte chunks XORed with row & 15 so that
// both operand reads are free of bank conflicts), once for all 128 rows.
// A wavefront computes the 16-key blocks that its own M-block lists and
// skips the others, so nothing is computed for a neighbour's tiles.
//
// Each buffer is filled while the other one is used: V(t) while S(t) is
// formed, K(t + 1) during the weights and O += V(t)^T P(t); two barriers a
// step.  64 KB of LDS and at most 128 registers (D = 128) keep two
// workgroups on a CU, four wavefronts on a SIMD.  Staging 128 rows' keys once
// is what lifts it off the L2: with every wavefront reading its own operands
// the same input takes 1.6 ms instead of 0.41.

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

constexpr int kStepKeys = 64;
constexpr int kUnitWaves = kF32UnitThreads / 64;  // of 16 rows
static_assert(kUnitWaves * kRows == kUnitRows, "a wavefront per 16 rows");
constexpr int kBufferWord3 = 0x00020000;  // gfx9-family raw buffer resource word 3

__device__ __forceinline__ f32x4 lds4(int addr) {
  return *reinterpret_cast<const lds_f32x4*>(static_cast<size_t>(addr));
}

// Global -> LDS, 16 bytes per lane from byte voff of the resource, landing
// at m0 + 16 * lane.
__device__ __forceinline__ void dma_b128(int m0, int voff, const i32x4& rs) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(m0), "v"(voff), "s"(rs)
               : "memory", "m0");
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// kDma: K and V start on a 16-byte line; else they are staged through registers
// (4,224 tokens, 32/8 heads, D = 128: T = 64 437 us by DMA / 429, T = 16 415 /
// 455; over the lists 1430 and 1246).
template <int T, int D, bool kDma>
__global__ __launch_bounds__(kF32UnitThreads, 4) void attn_f32_unit_kernel(WorkTables wt,
                                                                          AttnArgs a) {
  constexpr int kG = kStepKeys / T;          // tiles of a step
  constexpr int kC = D / 16, kVc = D / 64;
  constexpr int kRowB = D * 4;               // bytes of a staged row
  constexpr int kBuf = kStepKeys * kRowB;    // bytes of a staged K or V step
  constexpr int kDmaRows = 1024 / kRowB;     // rows of one DMA instruction
  constexpr int kDmas = 8 / kDmaRows;        // instructions of a wavefront's 8 rows
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * kBuf];

  const int4* __restrict__ rp = reinterpret_cast<const int4*>(
      wt.launch + (wt.by_chunks ? chunk_place(wt, blockIdx.x) : static_cast<int32_t>(blockIdx.x)));
  const int4 ra = rp[0];  // head, kv head, rank, slot
  const int4 rb = rp[1];  // first token and length of the two blocks
  const int4 rc = rp[2];  // step offset, step count
  const int h = ra.x, kvh = ra.y, slot = ra.w;
  const int nsteps = rc.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int i = lane & 15;
  const int g = lane >> 4;
  const int blk = wave >> 2;                 // 64-row block of the unit
  const int wq = wave & 3;                   // 16-row block of that
  const int qlen = (blk == 0 ? rb.z : rb.w) - kRows * wq;
  const int64_t qtok = static_cast<int64_t>(blk == 0 ? rb.x : rb.y) + kRows * wq;
  const float c2 = a.scale_log2;

  const int row_bytes = a.hkv * kRowB;
  const int lds = static_cast<int>(reinterpret_cast<size_t>((lds_float*)smem));
  // this wavefront's DMA rows 8 w .. 8 w + 7: lane -> row, physical chunk
  constexpr int kChunks = kRowB / 16;
  const int drow = lane / kChunks;
  const int off0 = (8 * wave + drow) * row_bytes +
                   (((lane % kChunks) ^ ((8 * wave & 15) + drow)) << 4);
  const int lds_dma = lds + 8 * wave * kRowB;
  auto dma = [&](int to, const void* base, int64_t row0, int len) {
    const unsigned long long ad =
        reinterpret_cast<unsigned long long>(base) +
        static_cast<unsigned long long>(row0 * row_bytes + static_cast<int64_t>(kvh) * kRowB);
    if constexpr (!kDma) {
      const char* src = reinterpret_cast<const char*>(ad);
#pragma unroll
      for (int it = 0; it < kDmas; ++it) {
        f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
        if (8 * wave + it * kDmaRows + drow < len)
          x = load4(reinterpret_cast<const float*>(src + (off0 ^ ((it * kDmaRows) << 4)) +
                                                   it * kDmaRows * row_bytes));
        *reinterpret_cast<lds_f32x4*>(static_cast<size_t>(to + it * 1024 + lane * 16)) = x;
      }
      return;
    }
    i32x4 rs = i32x4{static_cast<int>(static_cast<unsigned>(ad)),
                     static_cast<int>((ad >> 32) & 0xffff), (len - 1) * row_bytes + kRowB,
                     kBufferWord3};
    // uniform, which the compiler does not see: the DMA takes scalar registers
#pragma unroll
    for (int j = 0; j < 4; ++j) rs[j] = __builtin_amdgcn_readfirstlane(rs[j]);
#pragma unroll
    for (int it = 0; it < kDmas; ++it)
      dma_b128(to + it * 1024, (off0 ^ ((it * kDmaRows) << 4)) + it * kDmaRows * row_bytes, rs);
  };
  const int2* __restrict__ steps = wt.steps + rc.x;
  // T < 64: the first row of the tile that this wavefront's DMA rows are in
  const int* __restrict__ kvb = reinterpret_cast<const int*>(wt.kvb + rc.x) + (8 * wave) / T;
  struct Step {
    int x, info, row0;
  };
  auto fetch = [&](int t) {
    const int2 s = steps[t];
    Step st;
    st.x = __builtin_amdgcn_readfirstlane(s.x);
    st.info = __builtin_amdgcn_readfirstlane(s.y);
    st.row0 = kG > 1 ? __builtin_amdgcn_readfirstlane(kvb[4 * t]) : st.x;
    return st;
  };

  f32x4 qf[kC];
  {
    const float* q = static_cast<const float*>(a.q) +
                     ((qtok + min(i, max(qlen, 1) - 1)) * a.hq + h) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < kC; ++c) {
      qf[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (qlen > 0) qf[c] = load4(q + 16 * c);
    }
  }
  f32x4 o[4 * kVc];
#pragma unroll
  for (int d = 0; d < 4 * kVc; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mref = -INFINITY, lsum = 0.f;
  // operand reads: K row 16 kb + i, chunk 4 c + g; V row 16 kb + 4 g + r,
  // chunk 16 c + i
  const int ka = lds + i * kRowB + ((g ^ i) << 4);
  const int va = lds + kBuf + 4 * g * kRowB + ((i ^ (4 * g)) << 4);

  Step cur{0, 0, 0};
  if (nsteps > 0) {
    cur = fetch(0);
    dma(lds_dma, a.k, cur.row0, cur.info & kStepLenMask);
  }
  for (int t = 0; t < nsteps; ++t) {
    const int len = cur.info & kStepLenMask;
    wait_dma();
    __syncthreads();  // K(t) is there; V(t - 1) has been used
    dma(lds_dma + kBuf, a.v, cur.row0, len);
    const Step nxt = fetch(t + 1 < nsteps ? t + 1 : t);
    // the step's 16-key blocks that this wavefront's M-block lists
    const bool diag = (cur.info >> (kStepDiagShift + blk)) & 1;
    unsigned act = 0u;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const bool on =
          kG == 1 ? (cur.info >> (kStepListedShift + blk)) & 1
                  : (cur.x >> (kG * (kG * blk + kRows * wq / T) + kRows * kb / T)) & 1;
      if (on && kRows * kb < len && !(diag && kb > wq)) act |= 1u << kb;
    }
    f32x4 s[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
      if ((act >> kb) & 1u) {
#pragma unroll
        for (int c = 0; c < kC; ++c) {
          const f32x4 kf = lds4((ka ^ ((c & 3) << 6)) + (c >> 2) * 256 + kb * kRows * kRowB);
#pragma unroll
          for (int r = 0; r < 4; ++r) s[kb] = mfma(kf[r], qf[c][r], s[kb]);
        }
        if ((diag && kb == wq) || kRows * kb + kRows > len) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int key = kRows * kb + 4 * g + r;
            if (key >= len || (diag && key > kRows * wq + i)) s[kb][r] = -INFINITY;
          }
        }
      } else {
        s[kb] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      }
    }
    wait_dma();
    __syncthreads();  // V(t) is there; K(t) has been used
    if (t + 1 < nsteps) dma(lds_dma, a.k, nxt.row0, nxt.info & kStepLenMask);
    cur = nxt;
    if (act == 0u) continue;
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[kb][r]);
    float sum = 0.f;  // the step's weights
    rescale<D>(quad_max(mx) * c2, mref, lsum, sum, o);
    const float base = mref == -INFINITY ? 0.f : mref;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if (!((act >> kb) & 1u)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = exp2f(fmaf(s[kb][r], c2, -base));
        sum += p;
#pragma unroll
        for (int c = 0; c < kVc; ++c) {
          const f32x4 vf = lds4((va ^ (r << 4)) + (kRows * kb + r) * kRowB + c * 256);
#pragma unroll
          for (int d = 0; d < 4; ++d) o[4 * c + d] = mfma(vf[d], p, o[4 * c + d]);
        }
      }
    }
    lsum += sum;
  }

  lsum = quad_sum(lsum);
  if (i >= qlen) return;
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  float* dst = static_cast<float*>(a.out) + ((qtok + i) * a.hq + h) * D + 16 * g;
  if (slot >= 0) {
    // a piece: its normalised rows, their reference max and sum
    const int64_t srow = static_cast<int64_t>(slot) * kUnitRows + ((qtok + i) & (kUnitRows - 1));
    dst = static_cast<float*>(wt.part_o) + srow * D + 16 * g;
    if (g == 0) wt.part_ml[srow] = make_float2(mref, lsum);
  }
#pragma unroll
  for (int c = 0; c < kVc; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      store4(dst + 64 * c + 4 * r,
             f32x4{o[4 * c][r], o[4 * c + 1][r], o[4 * c + 2][r], o[4 * c + 3][r]} * inv);
}

// Merge the pieces of the split units: with M the largest reference max of
// the pieces that saw keys and w_p = l_p 2^(m_p - M), a row's output is
// sum w_p O_p / sum w_p.  Block 8 s + y takes rows 16 y .. + 15 of split
// unit s; thread t owns row t / 16 and dims 64 c + 4 (t % 16) .. + 3.
template <int D>
__global__ __launch_bounds__(256) void combine_kernel(WorkTables wt, AttnArgs a) {
  const int4 sp = wt.splits[blockIdx.x >> 3];  // {record of the first piece, first slot, slots}
  const WorkRec* __restrict__ rp = wt.rec + sp.x;
  const int row = (blockIdx.x & 7) * 16 + (threadIdx.x >> 4);
  const int blk = row >> 6, r = row & 63;
  if (r >= rp->len[blk]) return;
  const int64_t tok = rp->tok0[blk] + r;
  const int64_t srow = static_cast<int64_t>(sp.y) * kUnitRows + (tok & (kUnitRows - 1));
  const float2* ml = wt.part_ml + srow;
  float mx = -INFINITY;
  for (int p = 0; p < sp.z; ++p) {
    const float2 x = ml[static_cast<int64_t>(p) * kUnitRows];
    if (x.y > 0.f) mx = fmaxf(mx, x.x);
  }
  const int d0 = 4 * (threadIdx.x & 15);
  const float* po = static_cast<const float*>(wt.part_o) + srow * D + d0;
  f32x4 acc[D / 64];
#pragma unroll
  for (int c = 0; c < D / 64; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float wsum = 0.f;
#pragma unroll 2
  for (int p = 0; p < sp.z; ++p) {
    const float2 x = ml[static_cast<int64_t>(p) * kUnitRows];
    // a NaN sum (a NaN score) is kept
    const float w = x.y == 0.f ? 0.f : x.y * exp2f(x.x - mx);
    wsum += w;
#pragma unroll
    for (int c = 0; c < D / 64; ++c)
      acc[c] += load4(po + static_cast<int64_t>(p) * kUnitRows * D + 64 * c) * w;
  }
  const float inv = wsum > 0.f ? 1.f / wsum : wsum;
  float* dst = static_cast<float*>(a.out) + (tok * a.hq + rp->head) * D + d0;
#pragma unroll
  for (int c = 0; c < D / 64; ++c) store4(dst + 64 * c, acc[c] * inv);
}

template <int T, int D>
hipError_t launch_t(const PlanTables& pt, const WorkTables* wt, const AttnArgs& a,
                    hipStream_t stream) {
  const int tiles = kWaves * kRows / T;  // of a group
  const int64_t groups = (static_cast<int64_t>(pt.num_tiles) + tiles - 1) / tiles;
  const int64_t units = groups * pt.num_q_heads;
  if (units == 0) return hipSuccess;
  if (wt != nullptr && f32_units_fit(*wt) && (units >= kFewGroups || a.row_ptr == nullptr)) {
    // K and V rows are whole 16-byte chunks of the DMA only from a 16-byte line on
    if ((reinterpret_cast<uintptr_t>(a.k) | reinterpret_cast<uintptr_t>(a.v)) % 16 == 0)
      hipLaunchKernelGGL((attn_f32_unit_kernel<T, D, true>), dim3(wt->grid),
                         dim3(kF32UnitThreads), 0, stream, *wt, a);
    else
      hipLaunchKernelGGL((attn_f32_unit_kernel<T, D, false>), dim3(wt->grid),
                         dim3(kF32UnitThreads), 0, stream, *wt, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || wt->num_splits == 0) return e;
    hipLaunchKernelGGL((combine_kernel<D>), dim3(8 * wt->num_splits), dim3(256), 0, stream, *wt, a);
    return hipGetLastError();
  }
  const int64_t slots = (units + kNumXcd - 1) / kNumXcd * kNumXcd;
  // a grid holds fewer than 2^32 threads
  const int mode = slots * kWaves * 256 >= int64_t(1) << 32 ? kSplitNone
                   : units < kFewGroups                     ? kSplitAll
                                                            : kSplitQuery;
  hipLaunchKernelGGL((attn_f32_kernel<T, D>),
                     dim3(static_cast<unsigned>(mode == kSplitNone ? slots : slots * kWaves)),
                     dim3(256), 0, stream, pt, a, static_cast<int>(groups), mode);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const PlanTables& pt, const WorkTables* wt, const AttnArgs& a,
                           hipStream_t stream) {
  if (a.head_dim == 64) {
    if (a.tile == 16) return launch_t<16, 64>(pt, wt, a, stream);
    if (a.tile == 32) return launch_t<32, 64>(pt, wt, a, stream);
    if (a.tile == 64) return launch_t<64, 64>(pt, wt, a, stream);
  } else if (a.head_dim == 128) {
    if (a.tile == 16) return launch_t<16, 128>(pt, wt, a, stream);
    if (a.tile == 32) return launch_t<32, 128>(pt, wt, a, stream);
    if (a.tile == 64) return launch_t<64, 128>(pt, wt, a, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace sift
