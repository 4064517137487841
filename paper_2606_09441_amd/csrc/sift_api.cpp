// Host side of libsift: argument checks, the plan (tables derived from the
// prompt layout, Sections 4.3 and 5.1), the attention schedule, and the
// C ABI declared in include/sift.h.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <limits>
#include <list>
#include <memory>
#include <mutex>
#include <new>
#include <numeric>
#include <vector>

#include "sift.h"
#include "sift_internal.h"

namespace {


int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t la_nbytes(int64_t P) { return ceil_div(P * (P + 1), 16); }  // Section 4.3
int64_t ca_nbytes(int64_t P) { return ceil_div(P, 8); }             // Section 4.3

}  // namespace

struct sift_plan {
  int device = 0;
  sift_plan_info info{};
  // one device allocation holds every table, then the decode scratch
  void* dev = nullptr;
  size_t dev_bytes = 0;
  bool owns_dev = true;  // false: the caller's workspace (sift_sparse_prefill_ex)
  sift::PlanTables pt{};
  sift::WorkTables wt{};
  int32_t* counts = nullptr;   // [num_rows]
  int32_t* row_ptr = nullptr;  // [num_rows + 1]
  int32_t* col_idx = nullptr;  // [list_capacity]
  bool steps_paged = false;    // the last decode wrote page-pool rows into the steps
  bool steps_decoded = false;  // the steps are the last decode's (not merged caller lists)
  bool lists_own = false;      // the last decode wrote row_ptr and col_idx above
  unsigned long long decode_capture = 0;  // the graph capture it was part of (0: none, or
                                          // sift_plan_run's, whose attention follows it)
  bool unsorted = false;       // bf16 calls leave the schedule pass out (kFewChunked)
  hipStream_t last_stream = nullptr;  // the stream of the plan's last enqueued work
};

namespace {
// The attention takes the records themselves, chunk by chunk, and there is no
// schedule pass.
void run_in_place(sift::WorkTables& wt) {
  wt.launch = wt.rec;
  wt.hist = nullptr;
  wt.by_chunks = 1;
}

// Everything a decode or an attention launch needs from the plan.  sorted: the
// call decodes and attends in one, over fp32 inputs.  The records are good after
// any decode or merge, the launch slots only after one with a schedule pass,
// so an attention that does not follow its own decode never reads those of an
// unsorted plan.
sift::WorkTables work(const sift_plan* p, bool sorted) {
  sift::WorkTables wt = p->wt;
  if (p->unsorted && !sorted) run_in_place(wt);
  return wt;
}
}  // namespace

namespace {

sift_status check_tensor(const sift_tensor* t, int32_t tokens, int32_t heads, int32_t dim) {
  if (t == nullptr) return SIFT_E_NULL;
  if (t->data == nullptr && static_cast<int64_t>(t->tokens) * t->heads * t->head_dim > 0)
    return SIFT_E_NULL;
  if (t->dtype != SIFT_F32 && t->dtype != SIFT_BF16) return SIFT_E_UNSUPPORTED;
  if (t->tokens != tokens || t->heads != heads || t->head_dim != dim) return SIFT_E_SHAPE;
  return SIFT_OK;
}

sift_status check_device(const sift_plan* plan) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return SIFT_E_HIP;
  return dev == plan->device ? SIFT_OK : SIFT_E_PLAN;
}

// The graph capture that the stream takes part in, 0 if none.
unsigned long long capture_of(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(s, &status, &id) != hipSuccess) return 0;
  return status == hipStreamCaptureStatusActive ? id : 0;
}

// Shapes and dtypes of one call against the plan's sizes.
sift_status check_io(const sift_tensor* q, const sift_tensor* k, const sift_tensor* v,
                     const sift_tensor* out, int32_t tokens, int32_t hq, int32_t hkv, int32_t dim,
                     int32_t tile) {
  sift_status st;
  if ((st = check_tensor(q, tokens, hq, dim)) != SIFT_OK) return st;
  if ((st = check_tensor(k, tokens, hkv, dim)) != SIFT_OK) return st;
  if ((st = check_tensor(v, tokens, hkv, dim)) != SIFT_OK) return st;
  if ((st = check_tensor(out, tokens, hq, dim)) != SIFT_OK) return st;
  if (q->dtype != k->dtype || q->dtype != v->dtype) return SIFT_E_UNSUPPORTED;
  if (q->dtype == SIFT_BF16 && dim != 128) return SIFT_E_UNSUPPORTED;
  if (q->dtype == SIFT_F32 && (out->dtype != SIFT_F32 || tile > 64)) return SIFT_E_UNSUPPORTED;
  return SIFT_OK;
}

// Host tables of a validated layout.  The records per query head (list units,
// work units) are kept once per group, a run of M-blocks that every head has a
// unit of; write_unit_records, write_work_records and write_splits make the
// whole arrays, straight into the upload's memory.
struct Group {
  int32_t m0, nb, seg;
  bool query;
  int64_t cost;   // causal tiles of the group's last M-block: the union's length bound
  int64_t parts;  // pieces
  int64_t len;    // steps of a piece
  sift::WorkRec rec;  // its work units' records, but for the heads, slot and first step
};

// A write record of a group; its head, first step and first work unit open.
struct Part {
  sift::UnitRec rec;
  int64_t cost;       // tiles walked
  int64_t off, work;  // the group's first step and work unit, of one head
  int64_t unit_cost;
};

struct HostPlan {
  std::vector<int32_t> seg_tile0, seg_pages, seg_kind, seg_first, seg_la_off, seg_ca_off;
  std::vector<int32_t> tile_seg, tile_tok0, tile_len, tile_lo;
  std::vector<int32_t> tile_info;  // int4 per tile (see PlanTables::tile_info)
  std::vector<Group> groups;  // in locality order
  std::vector<Part> parts;    // longest walk first
  int32_t hkv = 0, group_heads = 0;
  int64_t num_units = 0;    // list units
  int64_t num_urec = 0;     // records of the decode write pass
  int64_t num_work = 0;     // work units
  int64_t num_splits = 0;   // split units
  int64_t head_steps = 0, head_work = 0;  // bound of the steps, and work units, of one head
  int64_t step_cap = 0;     // bound of all list units' steps
  int64_t chunk_size = 0;
  bool chunked = false;     // whether each chunk is whole kv heads
  bool scheduled = false;   // whether the decode has a schedule pass
  int64_t part_slots = 0;
  int64_t dense_tiles = 0;  // causal tiles of all prompts, one head
  int64_t la_bytes = 0, ca_bytes = 0;
  int32_t num_tokens = 0, num_segments = 0, num_tiles = 0;
};

// The list units' records in decode write order: longest walk first over all
// heads, units of one length in locality order.
void write_unit_records(const HostPlan& hp, sift::UnitRec* out) {
  const int64_t g = hp.group_heads;
  for (size_t i0 = 0; i0 < hp.parts.size();) {
    size_t i1 = i0;
    while (i1 < hp.parts.size() && hp.parts[i1].cost == hp.parts[i0].cost) ++i1;
    for (int32_t kv = 0; kv < hp.hkv; ++kv)
      for (size_t i = i0; i < i1; ++i)
        for (int64_t j = 0; j < g; ++j) {
          const Part& x = hp.parts[i];
          sift::UnitRec r = x.rec;
          r.head = static_cast<int32_t>(kv * g + j);
          r.step_off = static_cast<int32_t>(g * (kv * hp.head_steps + x.off) + j * x.unit_cost);
          r.work0 = static_cast<int32_t>(g * (kv * hp.head_work + x.work) + j * x.rec.nwork);
          *out++ = r;
        }
    i0 = i1;
  }
}

// The work units' records in locality order (work unit w is record w); the
// launch order is made on the device after each decode, from the step counts.
void write_work_records(const HostPlan& hp, sift::WorkRec* out) {
  int64_t slot = 0, off = 0;
  for (int32_t kv = 0; kv < hp.hkv; ++kv)
    for (const Group& x : hp.groups)
      for (int32_t j = 0; j < hp.group_heads; ++j) {
        for (int64_t i = 0; i < x.parts; ++i) {
          sift::WorkRec r = x.rec;
          r.head = kv * hp.group_heads + j;
          r.kv_head = kv;
          r.slot = x.parts > 1 ? static_cast<int32_t>(slot++) : -1;
          r.step_off = static_cast<int32_t>(off + i * x.len);
          *out++ = r;
        }
        off += x.cost;
      }
}

// The split units, int4 {record of the first piece, first slot, slots, 0}.
void write_splits(const HostPlan& hp, int32_t* out) {
  int64_t slot = 0, w = 0;
  for (int32_t kv = 0; kv < hp.hkv; ++kv)
    for (const Group& x : hp.groups)
      for (int32_t j = 0; j < hp.group_heads; ++j) {
        if (x.parts > 1) {
          const int32_t r[4] = {static_cast<int32_t>(w), static_cast<int32_t>(slot),
                                static_cast<int32_t>(x.parts), 0};
          std::memcpy(out, r, sizeof(r));
          out += 4;
          slot += x.parts;
        }
        w += x.parts;
      }
}

sift_status build_host_plan(const sift_layout* lay, int32_t hq, int32_t hkv, int32_t tile,
                            HostPlan& hp) {
  if (lay->num_prompts < 1) return SIFT_E_LAYOUT;
  if (lay->prompt_seg_ptr == nullptr || lay->seg_offsets == nullptr) return SIFT_E_NULL;
  const int32_t B = lay->num_prompts;
  const int32_t* psp = lay->prompt_seg_ptr;
  const int32_t* so = lay->seg_offsets;
  if (psp[0] != 0) return SIFT_E_LAYOUT;
  for (int32_t b = 0; b < B; ++b)
    if (psp[b + 1] <= psp[b]) return SIFT_E_LAYOUT;  // every prompt has its query segment
  const int32_t S = psp[B];
  if (so[0] != 0) return SIFT_E_LAYOUT;
  for (int32_t s = 0; s < S; ++s)
    if (so[s + 1] < so[s]) return SIFT_E_LAYOUT;
  hp.num_segments = S;
  hp.num_tokens = so[S];
  hp.seg_tile0.resize(S);
  hp.seg_pages.resize(S);
  hp.seg_kind.resize(S);
  hp.seg_first.resize(S);
  hp.seg_la_off.resize(S);
  hp.seg_ca_off.resize(S);
  int64_t tiles = 0, la_off = 0, ca_off = 0, dense = 0;
  const int64_t i32max = std::numeric_limits<int32_t>::max();
  for (int32_t b = 0; b < B; ++b) {
    const int64_t lo = tiles;
    for (int32_t s = psp[b]; s < psp[b + 1]; ++s) {
      const bool is_query = s == psp[b + 1] - 1;
      const int64_t len = static_cast<int64_t>(so[s + 1]) - so[s];
      if (!is_query && len < 1) return SIFT_E_LAYOUT;  // documents are not empty
      const int64_t P = ceil_div(len, tile);
      hp.seg_tile0[s] = static_cast<int32_t>(tiles);
      hp.seg_pages[s] = static_cast<int32_t>(P);
      hp.seg_kind[s] = is_query ? sift::kQuery : sift::kDocument;
      hp.seg_first[s] = psp[b];
      hp.seg_la_off[s] = static_cast<int32_t>(la_off);
      hp.seg_ca_off[s] = static_cast<int32_t>(ca_off);
      if (!is_query) {
        la_off += hq * la_nbytes(P);
        ca_off += hq * ca_nbytes(P);
        if (la_off > i32max || ca_off > i32max) return SIFT_E_CAPACITY;
      }
      // causal tiles of rows i = 0..P-1 of this segment: (tiles - lo) + i + 1
      dense += P * (tiles - lo) + P * (P + 1) / 2;
      tiles += P;
      if (tiles > i32max) return SIFT_E_CAPACITY;
    }
  }
  hp.num_tiles = static_cast<int32_t>(tiles);
  hp.la_bytes = la_off;
  hp.ca_bytes = ca_off;
  hp.dense_tiles = dense;
  if (dense * hq >= i32max) return SIFT_E_CAPACITY;  // int32 list offsets
  if (static_cast<int64_t>(tiles) * hq >= i32max) return SIFT_E_CAPACITY;

  hp.tile_seg.resize(tiles);
  hp.tile_tok0.resize(tiles);
  hp.tile_len.resize(tiles);
  hp.tile_lo.resize(tiles);
  hp.tile_info.resize(4 * tiles);
  for (int32_t b = 0; b < B; ++b) {
    const int32_t lo = hp.seg_tile0[psp[b]];
    for (int32_t s = psp[b]; s < psp[b + 1]; ++s) {
      const bool doc = hp.seg_kind[s] == sift::kDocument;
      const int32_t P = hp.seg_pages[s];
      for (int32_t i = 0; i < P; ++i) {
        const int32_t m = hp.seg_tile0[s] + i;
        hp.tile_seg[m] = s;
        hp.tile_tok0[m] = so[s] + i * tile;
        hp.tile_len[m] = std::min<int32_t>(tile, so[s + 1] - (so[s] + i * tile));
        hp.tile_lo[m] = lo;
        int32_t* ti = &hp.tile_info[4 * static_cast<int64_t>(m)];
        ti[0] = hp.tile_tok0[m];
        ti[1] = hp.tile_len[m];
        ti[2] = doc ? hp.seg_ca_off[s] + (i >> 3) : -1;
        ti[3] = doc ? static_cast<int32_t>(ca_nbytes(P) << 3) | (i & 7) : 0;
      }
    }
  }

  // Attention work units: (query head, M-blocks ub*p .. of a segment).  The
  // M-blocks of one document share the cross-attention part of their lists
  // (it depends on the key document only), so a unit stages each of those
  // key tiles once for all of its query rows.  The bf16 kernel works on
  // units of two 64-row blocks: 128 / T M-blocks of T <= 64 per unit (G =
  // 64 / T of them per kernel block), or one M-block of T = 128 (two halves,
  // each tile up to two steps).
  const int32_t halves = tile == 128 ? 2 : 1;
  const int32_t ub = tile == 128 ? 1 : sift::kUnitRows / tile;
  const int32_t G = tile < 64 ? 64 / tile : 1;
  std::vector<Group>& groups = hp.groups;
  for (int32_t s = 0; s < S; ++s) {
    const int32_t lo = hp.seg_tile0[hp.seg_first[s]];  // first tile of the prompt
    for (int32_t p = 0; p < hp.seg_pages[s]; p += ub) {
      const int32_t m0 = hp.seg_tile0[s] + p;
      const int32_t nb = std::min<int32_t>(ub, hp.seg_pages[s] - p);
      groups.push_back({m0, nb, s, hp.seg_kind[s] == sift::kQuery,
                        static_cast<int64_t>(m0 + nb - 1 - lo + 1) * halves, 1, 0, {}});
    }
  }
  // Units in locality order: kv head, then longest group first, then the
  // query heads of the kv group side by side (they read the same key tiles).
  // The launch cuts this order into kNumXcd equal chunks.  Where a cut falls
  // inside a kv head, its groups are first dealt to and fro into as many runs
  // as make every chunk a whole number of runs, so that each chunk gets long
  // and short groups alike: cut in order of length, one kv head's first chunk
  // held nearly twice the average work and its last one next to none.  us a
  // call, in order of length / dealt (T = 64, bf16): 66,048 tokens, 6/1 heads
  // 2427 / 1468; 16,640 tokens, 4/1 204 / 134, 8/2 262 / 196, 24/3 653 / 501;
  // 4,224 tokens, 8/1 60 / 57.  A multiple of 8 kv heads needs no deal.
  const int32_t g = hq / hkv;
  std::stable_sort(groups.begin(), groups.end(),
                   [](const Group& x, const Group& y) { return x.cost > y.cost; });
  const int64_t U = static_cast<int64_t>(groups.size()) * hq;
  if (U > i32max / 2) return SIFT_E_CAPACITY;
  const int32_t runs = sift::kNumXcd / std::gcd(sift::kNumXcd, hkv);
  if (runs > 1) {
    std::vector<Group> dealt;
    dealt.reserve(groups.size());
    for (int32_t r = 0; r < runs; ++r)
      for (size_t i = 0; i < groups.size(); ++i) {
        const int32_t at = static_cast<int32_t>(i % (2 * runs));
        if ((at < runs ? at : 2 * runs - 1 - at) == r) dealt.push_back(groups[i]);
      }
    groups.swap(dealt);
  }
  // Work units.  A query unit lists every tile of its prompt up to its last
  // M-block, so its list length is its cost.  The launch runs the longest
  // work units first (see WorkRec), so a unit only delays the end when it is
  // longer than the work per workgroup slot; a query unit is cut into pieces
  // of at most `piece` steps, piece = that work's lower bound (the query
  // units' steps plus one diagonal step per document M-block, over
  // kSlots resident workgroups), at least kMinPiece.  The piece length
  // doubles until at most kMaxSlots partial slots are needed.
  constexpr int64_t kMaxSlots = 4096;
  constexpr int64_t kMinPiece = 32;
  constexpr int64_t kSlots = 512;  // 256 CUs x 2 resident attention workgroups
  int64_t lower = 0, steps = 0;
  for (const Group& x : groups) {
    lower += hq * (x.query ? x.cost : x.nb);
    steps += hq * x.cost;
    if (steps > i32max) return SIFT_E_CAPACITY;
  }
  hp.num_units = U;
  hp.step_cap = steps;
  int64_t piece = std::max<int64_t>(kMinPiece, (lower + kSlots - 1) / kSlots);
  auto slots_for = [&](int64_t pc) {
    int64_t n = 0;
    for (const Group& x : groups)
      if (x.query && x.cost > pc) n += hq * ((x.cost + pc - 1) / pc);
    return n;
  };
  while (slots_for(piece) > kMaxSlots) piece *= 2;
  int64_t work = 0, split = 0;  // of one head: work units, partial slots
  hp.num_splits = 0;
  for (Group& x : groups) {
    x.parts = x.query && x.cost > piece ? (x.cost + piece - 1) / piece : 1;
    x.len = (x.cost + x.parts - 1) / x.parts;
    work += x.parts;
    if (x.parts > 1) {
      split += x.parts;
      hp.num_splits += hq;
    }
  }
  const int64_t W = work * hq;
  if (W > i32max / 2) return SIFT_E_CAPACITY;
  hp.num_work = W;
  hp.part_slots = split * hq;
  hp.hkv = hkv;
  hp.group_heads = g;
  hp.head_steps = hq > 0 ? steps / hq : 0;
  hp.head_work = work;
  // Records of the decode write pass: one per unit, except that at T < 64 a
  // query unit's walk (segment by segment over its prompt, in steps of G
  // adjacent tiles) is cut into parts of whole segments of about kPartTiles
  // tiles, one wavefront each.  They run longest walk first over all heads,
  // so that no long walk starts late.
  constexpr int64_t kPartTiles = 256;
  std::vector<Part>& parts = hp.parts;
  {
    int64_t off = 0, w0 = 0;
    for (Group& x : groups) {
      const int32_t m0 = x.m0, sg = x.seg;
      sift::UnitRec r{};
      r.m0 = m0;
      r.nb = x.nb;
      r.seg = sg;
      r.lo = hp.tile_lo[m0];
      r.sd0 = hp.seg_tile0[sg];
      r.pages = hp.seg_pages[sg];
      r.la_off = hp.seg_la_off[sg];
      r.nwork = static_cast<int32_t>(x.parts);
      r.plen = static_cast<int32_t>(x.len);
      r.flags = (x.query ? sift::kUnitQuery : 0) | ((hp.tile_len[m0] > 64 ? 3 : 1) << 1);
      r.part_t0 = r.lo;
      r.part_t1 = m0 + x.nb;
      r.part_skip = 0;
      if (!(x.query && G > 1)) {
        r.flags |= sift::kUnitFirstPart | sift::kUnitLastPart;
        parts.push_back({r, x.cost, off, w0, x.cost});
      } else {
        // segment d's tiles walked by the unit, and its steps (groups of G)
        const int32_t mlast = m0 + r.nb - 1;
        auto tiles = [&](int32_t d) {
          return d < sg ? hp.seg_pages[d] : mlast - hp.seg_tile0[sg] + 1;
        };
        int32_t skip = 0;
        const int32_t first = hp.seg_first[sg];
        for (int32_t d0 = first; d0 <= sg;) {
          int32_t d1 = d0;
          int64_t t = 0, n = 0;
          while (d1 <= sg && (d1 == d0 || t + tiles(d1) <= kPartTiles)) {
            t += tiles(d1);
            n += (tiles(d1) + G - 1) / G;
            ++d1;
          }
          sift::UnitRec p = r;
          p.part_t0 = hp.seg_tile0[d0];
          p.part_t1 = d1 <= sg ? hp.seg_tile0[d1] : mlast + 1;
          p.part_skip = skip;
          if (d0 == first) p.flags |= sift::kUnitFirstPart;
          if (d1 == sg + 1) p.flags |= sift::kUnitLastPart;
          parts.push_back({p, t, off, w0, x.cost});
          skip += static_cast<int32_t>(n);
          d0 = d1;
        }
      }
      off += x.cost;
      w0 += x.parts;
      sift::WorkRec& wr = x.rec;
      if (halves == 1) {
        // kernel block b: M-blocks m0 + G b .. m0 + G b + G - 1 of the unit
        const int32_t blocks = (x.nb + G - 1) / G;
        for (int b = 0; b < blocks; ++b) {
          wr.tok0[b] = hp.tile_tok0[m0 + G * b];
          wr.len[b] = 0;
          for (int32_t m = m0 + G * b; m < std::min(m0 + x.nb, m0 + G * b + G); ++m)
            wr.len[b] += hp.tile_len[m];
        }
      } else {  // one M-block of T = 128: two kernel blocks of 64 rows
        const int32_t len = hp.tile_len[m0];
        wr.tok0[0] = hp.tile_tok0[m0];
        wr.len[0] = std::min<int32_t>(len, 64);
        wr.tok0[1] = len > 64 ? hp.tile_tok0[m0] + 64 : 0;
        wr.len[1] = len > 64 ? len - 64 : 0;
      }
    }
  }
  hp.num_urec = static_cast<int64_t>(parts.size()) * hq;
  if (hp.num_urec > i32max / 2) return SIFT_E_CAPACITY;
  std::stable_sort(parts.begin(), parts.end(),
                   [](const Part& x, const Part& y) { return x.cost > y.cost; });
  hp.chunk_size = (W + sift::kNumXcd - 1) / sift::kNumXcd;
  return SIFT_OK;
}

}  // namespace

extern "C" {

const char* sift_status_string(int32_t status) {
  switch (status) {
    case SIFT_OK: return "ok";
    case SIFT_E_NULL: return "a required pointer is NULL";
    case SIFT_E_SHAPE: return "tensor shapes do not match each other or the layout";
    case SIFT_E_LAYOUT: return "malformed prompt layout";
    case SIFT_E_UNSUPPORTED: return "tile size, head size or dtype not supported";
    case SIFT_E_CAPACITY: return "a buffer or index range is too small";
    case SIFT_E_HIP: return "a HIP runtime call failed";
    case SIFT_E_PLAN: return "the plan does not match the arguments or the device";
    default: return "unknown status";
  }
}

}  // extern "C"

namespace {

// Pinned host staging for stream-ordered uploads of plan tables.  A buffer
// is handed out to one call at a time; after the call has enqueued its copy
// it records an event, and the buffer is reused once that event has
// completed (the copy has read it).  No call waits: one that finds every
// buffer busy makes another, so there are at most as many as calls were queued
// at once (the copies of a program's own unfinished work).  Those beyond
// kKeptStaging per device go back when a plan is destroyed, which waits for
// the device anyway to free its memory.
struct StagingBuf {
  int device;
  void* host;
  size_t cap;
  hipEvent_t done;
  bool taken;
};
constexpr size_t kKeptStaging = 64;
std::mutex g_staging_mu;
std::list<StagingBuf> g_staging;  // addresses stay valid

// A pinned buffer of at least n bytes on the current device, not in use.
sift_status staging_acquire(size_t n, StagingBuf** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return SIFT_E_HIP;
  {
    std::lock_guard<std::mutex> lock(g_staging_mu);
    for (StagingBuf& b : g_staging) {
      if (b.taken || b.device != dev || b.cap < n) continue;
      const hipError_t q = hipEventQuery(b.done);
      if (q == hipErrorNotReady) continue;
      if (q != hipSuccess) return SIFT_E_HIP;
      b.taken = true;
      *out = &b;
      return SIFT_OK;
    }
  }
  size_t cap = 1 << 16;
  while (cap < n) cap <<= 1;
  std::list<StagingBuf> made{{dev, nullptr, cap, nullptr, true}};
  StagingBuf& b = made.front();
  if (hipHostMalloc(&b.host, cap, hipHostMallocDefault) != hipSuccess) return SIFT_E_HIP;
  if (hipEventCreateWithFlags(&b.done, hipEventDisableTiming) != hipSuccess) {
    (void)hipHostFree(b.host);
    return SIFT_E_HIP;
  }
  std::lock_guard<std::mutex> lock(g_staging_mu);
  g_staging.splice(g_staging.end(), made);
  *out = &b;
  return SIFT_OK;
}

// Give back the device's idle buffers beyond kKeptStaging.  Freeing pinned
// memory may wait for the device.
void staging_trim(int dev) {
  std::list<StagingBuf> spare;
  {
    std::lock_guard<std::mutex> lock(g_staging_mu);
    size_t held = 0;
    for (const StagingBuf& b : g_staging) held += b.device == dev ? 1 : 0;
    for (auto it = g_staging.begin(); it != g_staging.end() && held > kKeptStaging;) {
      const auto b = it++;
      if (b->device != dev || b->taken || hipEventQuery(b->done) != hipSuccess) continue;
      spare.splice(spare.end(), g_staging, b);
      --held;
    }
  }
  for (StagingBuf& b : spare) {
    (void)hipEventDestroy(b.done);
    (void)hipHostFree(b.host);
  }
}

// Hand a buffer back; with record, once the copies enqueued on the stream so
// far are done.
sift_status staging_release(StagingBuf* b, hipStream_t stream, bool record) {
  std::lock_guard<std::mutex> lock(g_staging_mu);
  b->taken = false;
  if (record && hipEventRecord(b->done, stream) != hipSuccess) return SIFT_E_HIP;
  return SIFT_OK;
}

}  // namespace

namespace sift {

hipError_t upload_staged(void* dst, size_t n, hipStream_t stream,
                         const std::function<void(uint8_t*)>& fill) {
  StagingBuf* b = nullptr;
  if (staging_acquire(n, &b) != SIFT_OK) return hipErrorUnknown;
  fill(static_cast<uint8_t*>(b->host));
  const hipError_t e = hipMemcpyAsync(dst, b->host, n, hipMemcpyHostToDevice, stream);
  if (staging_release(b, stream, e == hipSuccess) != SIFT_OK && e == hipSuccess)
    return hipErrorUnknown;
  return e;
}

}  // namespace sift

namespace {

// How the plan's tables reach the device.
enum class Upload {
  kBlocking,   // hipMemcpy into the plan's own hipMalloc (sift_plan_create)
  kStaged,     // hipMemcpyAsync on `stream` from pinned staging: no host wait
  kPageable,   // hipMemcpyAsync on `stream` from host memory, then a wait for
               // `stream` (no allocation at all)
};

// A checked layout's tables, and where each goes in the plan's device memory:
// the tables, then the schedule's bucket sizes and the attention's
// redo flag (zero: uploaded with the tables, and left so by every pass that
// uses them), then the decode and merge scratch.
struct PlanImage {
  HostPlan hp;
  int32_t hq, hkv, head_dim, tile;
  // byte offsets of the tables
  size_t seg_tile0, seg_pages, seg_kind, seg_first, seg_la, seg_ca;
  size_t tile_seg, tile_tok0, tile_len, tile_lo, tile_info;
  size_t urec, rec, launch, splits, hist;
  size_t upload;  // bytes of the tables
  // of the scratch
  size_t counts, segbase, headtot, camark, segcross, crosscol, crossrows, rowptr, col, steps, kvb;
  size_t part_o, part_lo, part_ml;
  size_t total;
};

// the schedule's bucket sizes, the bf16 attention's redo flag and counters,
// the decode's finished-block count: zeros, uploaded with the tables
constexpr size_t kHistWords = sift::kNumXcd * sift::kSchedBuckets + 4 + sift::kNumXcd;

sift_status make_image(const sift_layout* layout, int32_t num_q_heads, int32_t num_kv_heads,
                       int32_t head_dim, int32_t tile, PlanImage& im) {
  if (layout == nullptr) return SIFT_E_NULL;
  if (num_q_heads < 1 || num_kv_heads < 1 || num_q_heads % num_kv_heads != 0) return SIFT_E_SHAPE;
  if (head_dim != 64 && head_dim != 128) return SIFT_E_UNSUPPORTED;
  if (tile != 16 && tile != 32 && tile != 64 && tile != 128) return SIFT_E_UNSUPPORTED;
  HostPlan& hp = im.hp;
  sift_status st = build_host_plan(layout, num_q_heads, num_kv_heads, tile, hp);
  if (st != SIFT_OK) return st;
  im.hq = num_q_heads;
  im.hkv = num_kv_heads;
  im.head_dim = head_dim;
  im.tile = tile;
  size_t at = 0;
  auto place = [&at](size_t n) {
    const size_t off = (at + 255) & ~size_t(255);
    at = off + n;
    return off;
  };
  auto ints = [&](const std::vector<int32_t>& v) { return place(v.size() * sizeof(int32_t)); };
  im.seg_tile0 = ints(hp.seg_tile0);
  im.seg_pages = ints(hp.seg_pages);
  im.seg_kind = ints(hp.seg_kind);
  im.seg_first = ints(hp.seg_first);
  im.seg_la = ints(hp.seg_la_off);
  im.seg_ca = ints(hp.seg_ca_off);
  im.tile_seg = ints(hp.tile_seg);
  im.tile_tok0 = ints(hp.tile_tok0);
  im.tile_len = ints(hp.tile_len);
  im.tile_lo = ints(hp.tile_lo);
  im.tile_info = ints(hp.tile_info);
  im.urec = place(hp.num_urec * sizeof(sift::UnitRec));
  hp.chunked = num_kv_heads % sift::kNumXcd == 0;
  hp.scheduled = hp.num_work > sift::kFewUnits;
  const int64_t slots = hp.chunk_size * sift::kNumXcd;
  im.rec = place(slots * sizeof(sift::WorkRec));  // counts and first steps: by decode
  im.launch = place((hp.scheduled ? slots : 0) * sizeof(sift::WorkRec));  // by the schedule pass
  im.splits = place(hp.num_splits * 4 * sizeof(int32_t));
  im.hist = place(kHistWords * sizeof(int32_t));
  im.upload = at;
  const int64_t rows = static_cast<int64_t>(hp.num_tiles) * num_q_heads;
  const int64_t segs = static_cast<int64_t>(hp.num_segments) * num_q_heads;
  const int64_t cap = hp.dense_tiles * num_q_heads;
  im.counts = place(rows * 4);
  im.segbase = place(segs * 4);
  im.headtot = place(static_cast<int64_t>(num_q_heads) * 4);
  im.camark = place(rows);
  im.segcross = place(segs * 4);
  im.crosscol = place(rows * 4);
  im.crossrows = place(rows * 8);
  im.rowptr = place((rows + 1) * 4);
  im.col = place(std::max<int64_t>(cap, 1) * 4);
  // steps: the units' lists, plus a few entries read (never used) past the end
  // (the lists' total length bound: one step per listed tile at T <= 64, up
  // to two at T = 128); per-step K/V row bases at T < 64 only
  const int64_t step_room = std::max<int64_t>(hp.step_cap, 1) + 8;
  im.steps = place(step_room * 8);
  im.kvb = place(tile < 64 ? step_room * 16 : 0);
  const int64_t slot_rows = hp.part_slots * sift::kUnitRows;
  // the pieces' outputs: fp32, or bf16 plus the bf16 of its rounding error
  im.part_o = place(slot_rows * head_dim * 4);
  im.part_lo = place(slot_rows * head_dim * 2);
  im.part_ml = place(std::max<int64_t>(slot_rows, 1) * 8);
  im.total = at;
  return SIFT_OK;
}

// The tables, im.upload bytes.
void write_tables(const PlanImage& im, uint8_t* out) {
  const HostPlan& hp = im.hp;
  auto ints = [out](size_t off, const std::vector<int32_t>& v) {
    if (!v.empty()) std::memcpy(out + off, v.data(), v.size() * sizeof(int32_t));
  };
  ints(im.seg_tile0, hp.seg_tile0);
  ints(im.seg_pages, hp.seg_pages);
  ints(im.seg_kind, hp.seg_kind);
  ints(im.seg_first, hp.seg_first);
  ints(im.seg_la, hp.seg_la_off);
  ints(im.seg_ca, hp.seg_ca_off);
  ints(im.tile_seg, hp.tile_seg);
  ints(im.tile_tok0, hp.tile_tok0);
  ints(im.tile_len, hp.tile_len);
  ints(im.tile_lo, hp.tile_lo);
  ints(im.tile_info, hp.tile_info);
  write_unit_records(hp, reinterpret_cast<sift::UnitRec*>(out + im.urec));
  write_work_records(hp, reinterpret_cast<sift::WorkRec*>(out + im.rec));
  // launch slots start empty (one M-block of no rows, no steps); the
  // schedule pass fills those of the work units.  Without one the records
  // are the launch slots, and those past the work units stay empty
  sift::WorkRec empty{};
  empty.slot = -1;
  const int64_t slots = hp.chunk_size * sift::kNumXcd;
  std::fill_n(reinterpret_cast<sift::WorkRec*>(out + im.rec) + hp.num_work, slots - hp.num_work,
              empty);
  if (hp.scheduled)
    std::fill_n(reinterpret_cast<sift::WorkRec*>(out + im.launch), slots, empty);
  write_splits(hp, reinterpret_cast<int32_t*>(out + im.splits));
  std::memset(out + im.hist, 0, kHistWords * sizeof(int32_t));
}

// The plan of an image.  Its device memory: with ws == nullptr a hipMalloc of
// its own, else ws (ws_bytes, 256-byte aligned): the caller's workspace,
// stream-ordered scratch or static scratch, written on `stream` as `up` says.
sift_status create_plan(const PlanImage& im, void* ws, size_t ws_bytes, hipStream_t stream,
                        Upload up, sift_plan** plan_out) {
  if (plan_out == nullptr) return SIFT_E_NULL;
  *plan_out = nullptr;
  const HostPlan& hp = im.hp;
  const size_t total = im.total;
  if (ws != nullptr) {
    if (ws_bytes < total) return SIFT_E_CAPACITY;
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return SIFT_E_UNSUPPORTED;
  }
  sift_plan* plan = new (std::nothrow) sift_plan();
  if (plan == nullptr) return SIFT_E_HIP;
  if (hipGetDevice(&plan->device) != hipSuccess) {
    delete plan;
    return SIFT_E_HIP;
  }
  auto fail = [plan]() {
    if (plan->owns_dev && plan->dev != nullptr) (void)hipFree(plan->dev);
    delete plan;
    return SIFT_E_HIP;
  };
  plan->dev_bytes = total;
  if (ws != nullptr) {
    plan->dev = ws;
    plan->owns_dev = false;
    plan->last_stream = stream;
  } else if (hipMalloc(&plan->dev, total) != hipSuccess) {
    return fail();
  }
  if (up == Upload::kStaged) {
    // from pinned staging: the call returns without waiting
    if (sift::upload_staged(plan->dev, im.upload, stream,
                            [&im](uint8_t* out) { write_tables(im, out); }) != hipSuccess)
      return fail();
  } else {
    std::unique_ptr<uint8_t[]> host(new (std::nothrow) uint8_t[im.upload]);
    if (host == nullptr) return fail();
    write_tables(im, host.get());
    if (up == Upload::kBlocking) {
      if (hipMemcpy(plan->dev, host.get(), im.upload, hipMemcpyHostToDevice) != hipSuccess)
        return fail();
    } else {
      // host memory: it must outlive the copy, so wait for the stream
      if (hipMemcpyAsync(plan->dev, host.get(), im.upload, hipMemcpyHostToDevice, stream) !=
              hipSuccess ||
          hipStreamSynchronize(stream) != hipSuccess)
        return fail();
    }
  }
  auto P = [plan](size_t off) {
    return reinterpret_cast<int32_t*>(static_cast<uint8_t*>(plan->dev) + off);
  };
  plan->pt.seg_tile0 = P(im.seg_tile0);
  plan->pt.seg_pages = P(im.seg_pages);
  plan->pt.seg_kind = P(im.seg_kind);
  plan->pt.seg_first = P(im.seg_first);
  plan->pt.seg_la_off = P(im.seg_la);
  plan->pt.seg_ca_off = P(im.seg_ca);
  plan->pt.tile_seg = P(im.tile_seg);
  plan->pt.tile_tok0 = P(im.tile_tok0);
  plan->pt.tile_len = P(im.tile_len);
  plan->pt.tile_lo = P(im.tile_lo);
  plan->pt.tile_info = reinterpret_cast<const int4*>(P(im.tile_info));
  plan->pt.tile = im.tile;
  plan->pt.halves = im.tile == 128 ? 2 : 1;
  plan->pt.group = im.tile < 64 ? 64 / im.tile : 1;
  plan->pt.num_tiles = hp.num_tiles;
  plan->pt.num_segments = hp.num_segments;
  plan->pt.num_q_heads = im.hq;
  plan->wt.rec = reinterpret_cast<sift::WorkRec*>(P(im.rec));
  plan->wt.launch = hp.scheduled ? reinterpret_cast<sift::WorkRec*>(P(im.launch)) : plan->wt.rec;
  plan->wt.hist = hp.scheduled ? P(im.hist) : nullptr;
  plan->wt.urec = reinterpret_cast<const sift::UnitRec*>(P(im.urec));
  plan->wt.steps = reinterpret_cast<int2*>(P(im.steps));
  plan->wt.kvb = im.tile < 64 ? reinterpret_cast<int4*>(P(im.kvb)) : nullptr;
  plan->wt.splits = reinterpret_cast<const int4*>(P(im.splits));
  plan->wt.part_o = static_cast<void*>(P(im.part_o));
  plan->wt.part_lo = static_cast<void*>(P(im.part_lo));
  plan->wt.part_ml = reinterpret_cast<float2*>(P(im.part_ml));
  plan->wt.redo = P(im.hist) + sift::kNumXcd * sift::kSchedBuckets;
  plan->wt.decode_done = plan->wt.redo + 3;
  plan->wt.sched_done = plan->wt.redo + 4;
  plan->wt.seg_base = P(im.segbase);
  plan->wt.head_tot = P(im.headtot);
  plan->wt.ca_mark = reinterpret_cast<uint8_t*>(P(im.camark));
  plan->wt.seg_cross = P(im.segcross);
  plan->wt.cross_col = P(im.crosscol);
  plan->wt.cross_rows = reinterpret_cast<int2*>(P(im.crossrows));
  plan->wt.num_units = static_cast<int32_t>(hp.num_units);
  plan->wt.num_urec = static_cast<int32_t>(hp.num_urec);
  plan->wt.num_work = static_cast<int32_t>(hp.num_work);
  plan->wt.num_splits = static_cast<int32_t>(hp.num_splits);
  plan->wt.chunk_size = static_cast<int32_t>(hp.chunk_size);
  plan->wt.sched_blocks = static_cast<int32_t>(
      std::min<int64_t>(8, std::max<int64_t>(1, ceil_div(hp.chunk_size, sift::kSchedPerBlock))));
  plan->wt.grid = static_cast<int32_t>(hp.chunk_size * sift::kNumXcd);
  if (hp.chunked && !hp.scheduled) run_in_place(plan->wt);
  plan->unsorted = im.hkv == sift::kNumXcd && hp.scheduled &&
                   hp.num_work <= sift::kFewChunked && im.tile >= 64 && im.head_dim == 128;
  plan->counts = P(im.counts);
  plan->row_ptr = P(im.rowptr);
  plan->col_idx = P(im.col);

  sift_plan_info& in = plan->info;
  in.num_tokens = hp.num_tokens;
  in.num_segments = hp.num_segments;
  in.num_tiles = hp.num_tiles;
  in.num_q_heads = im.hq;
  in.num_kv_heads = im.hkv;
  in.head_dim = im.head_dim;
  in.tile = im.tile;
  in.num_work_units = static_cast<int32_t>(hp.num_work);
  in.num_rows = static_cast<int64_t>(hp.num_tiles) * im.hq;
  in.list_capacity = hp.dense_tiles * im.hq;
  in.la_bytes = hp.la_bytes;
  in.ca_bytes = hp.ca_bytes;
  in.scratch_bytes = static_cast<int64_t>(total);
  *plan_out = plan;
  return SIFT_OK;
}

// Arguments of the one-shot forms, checked on the host before anything is
// enqueued; im receives the image of their plan.
sift_status check_prefill(const sift_tensor* q, const sift_tensor* k, const sift_tensor* v,
                          const sift_layout* layout, const uint8_t* la, const uint8_t* ca,
                          int32_t tile, const sift_tensor* out, PlanImage& im) {
  if (q == nullptr || k == nullptr || v == nullptr || out == nullptr || layout == nullptr)
    return SIFT_E_NULL;
  if (q->heads < 1 || k->heads < 1 || q->heads % k->heads != 0) return SIFT_E_SHAPE;
  sift_status st = make_image(layout, q->heads, k->heads, q->head_dim, tile, im);
  if (st != SIFT_OK) return st;
  st = check_io(q, k, v, out, im.hp.num_tokens, q->heads, k->heads, q->head_dim, tile);
  if (st != SIFT_OK) return st;
  if (im.hp.la_bytes > 0 && la == nullptr) return SIFT_E_NULL;
  if (im.hp.ca_bytes > 0 && ca == nullptr) return SIFT_E_NULL;
  return SIFT_OK;
}

// Scratch for sift_sparse_prefill_static: one array per GPU, held from the
// library's load on that GPU until the process ends.  Host code never uses
// the array's name as an address: each device's address is taken once with
// hipGetSymbolAddress, with that device current, and kept here.
constexpr size_t kStaticScratchBytes = size_t(256) << 20;
__device__ __align__(256) uint8_t scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::once_flag g_scratch_once[kMaxDevices];
void* g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};

// The current device's address of the scratch array.
sift_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return SIFT_E_HIP;
  if (dev < 0 || dev >= kMaxDevices) return SIFT_E_UNSUPPORTED;
  std::call_once(g_scratch_once[dev], [dev]() {
    g_scratch_err[dev] = hipGetSymbolAddress(&g_scratch_ptr[dev], HIP_SYMBOL(scratch));
  });
  if (g_scratch_err[dev] != hipSuccess || g_scratch_ptr[dev] == nullptr) return SIFT_E_HIP;
  *out = g_scratch_ptr[dev];
  return SIFT_OK;
}

// Plans made only to decode lists: the lists do not depend on the kv heads
// or the head size, so the smallest attention scratch is taken.
constexpr int32_t kDecodeKvHeads = 1;
constexpr int32_t kDecodeHeadDim = 64;

}  // namespace

extern "C" {

sift_status sift_plan_create(const sift_layout* layout, int32_t num_q_heads,
                             int32_t num_kv_heads, int32_t head_dim, int32_t tile,
                             sift_plan** plan_out) {
  if (plan_out == nullptr) return SIFT_E_NULL;
  *plan_out = nullptr;
  PlanImage im;
  const sift_status st = make_image(layout, num_q_heads, num_kv_heads, head_dim, tile, im);
  if (st != SIFT_OK) return st;
  return create_plan(im, nullptr, 0, nullptr, Upload::kBlocking, plan_out);
}

sift_status sift_workspace_bytes(const sift_layout* layout, int32_t num_q_heads,
                                 int32_t num_kv_heads, int32_t head_dim, int32_t tile,
                                 size_t* bytes) {
  if (bytes == nullptr) return SIFT_E_NULL;
  PlanImage im;
  const sift_status st = make_image(layout, num_q_heads, num_kv_heads, head_dim, tile, im);
  if (st == SIFT_OK) *bytes = im.total;
  return st;
}

sift_status sift_plan_destroy(sift_plan* plan) {
  if (plan == nullptr) return SIFT_OK;
  sift_status st = SIFT_OK;
  if (plan->dev != nullptr && plan->owns_dev) {
    // the plan's last work may still read its memory
    if (hipStreamSynchronize(plan->last_stream) != hipSuccess) st = SIFT_E_HIP;
    if (hipFree(plan->dev) != hipSuccess) st = SIFT_E_HIP;
    staging_trim(plan->device);
  }
  delete plan;
  return st;
}

sift_status sift_plan_exact_passes(const sift_plan* plan, int64_t* count) {
  if (plan == nullptr || count == nullptr) return SIFT_E_NULL;
  if (check_device(plan) != SIFT_OK) return SIFT_E_PLAN;
  int32_t n = 0;
  if (hipMemcpyAsync(&n, plan->wt.redo + 2, sizeof(n), hipMemcpyDeviceToHost,
                     plan->last_stream) != hipSuccess ||
      hipStreamSynchronize(plan->last_stream) != hipSuccess)
    return SIFT_E_HIP;
  *count = n;
  return SIFT_OK;
}

sift_status sift_plan_get_info(const sift_plan* plan, sift_plan_info* info) {
  if (plan == nullptr || info == nullptr) return SIFT_E_NULL;
  *info = plan->info;
  return SIFT_OK;
}

static sift_status decode_lists(sift_plan* plan, const uint8_t* local_bitmap,
                                const uint8_t* cross_bitmap, int32_t* row_ptr, int32_t* col_idx,
                                int64_t col_capacity, bool sorted, void* stream) {
  if (plan == nullptr || row_ptr == nullptr) return SIFT_E_NULL;
  if (plan->info.la_bytes > 0 && local_bitmap == nullptr) return SIFT_E_NULL;
  if (plan->info.ca_bytes > 0 && cross_bitmap == nullptr) return SIFT_E_NULL;
  if (plan->info.list_capacity > 0 && col_idx == nullptr) return SIFT_E_NULL;
  if (col_capacity < plan->info.list_capacity) return SIFT_E_CAPACITY;
  sift_status st = check_device(plan);
  if (st != SIFT_OK) return st;
  const hipError_t e = sift::launch_decode(plan->pt, work(plan, sorted), local_bitmap,
                                           cross_bitmap, plan->counts, row_ptr, col_idx,
                                           sift::KvPages{nullptr, 0},
                                           static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return SIFT_E_HIP;
  plan->steps_paged = false;
  plan->steps_decoded = true;
  plan->lists_own = row_ptr == plan->row_ptr;
  plan->decode_capture = 0;
  plan->last_stream = static_cast<hipStream_t>(stream);
  return SIFT_OK;
}

sift_status sift_plan_decode_tiles(sift_plan* plan, const uint8_t* local_bitmap,
                                   const uint8_t* cross_bitmap, int32_t* row_ptr,
                                   int32_t* col_idx, int64_t col_capacity, void* stream) {
  const sift_status st =
      decode_lists(plan, local_bitmap, cross_bitmap, row_ptr, col_idx, col_capacity, false, stream);
  if (st == SIFT_OK) plan->decode_capture = capture_of(static_cast<hipStream_t>(stream));
  return st;
}

sift_status sift_plan_decode(sift_plan* plan, const uint8_t* local_bitmap,
                             const uint8_t* cross_bitmap, void* stream) {
  if (plan == nullptr) return SIFT_E_NULL;
  return sift_plan_decode_tiles(plan, local_bitmap, cross_bitmap, plan->row_ptr, plan->col_idx,
                                plan->info.list_capacity, stream);
}

sift_status sift_sparse_attention(sift_plan* plan, const sift_tensor* q, const sift_tensor* k,
                                  const sift_tensor* v, const int32_t* row_ptr,
                                  const int32_t* col_idx, int64_t col_capacity,
                                  float softmax_scale, sift_tensor* out, void* stream) {
  if (plan == nullptr || row_ptr == nullptr) return SIFT_E_NULL;
  const sift_plan_info& in = plan->info;
  sift_status st = check_io(q, k, v, out, in.num_tokens, in.num_q_heads, in.num_kv_heads,
                            in.head_dim, in.tile);
  if (st != SIFT_OK) return st;
  if (col_capacity < 0) return SIFT_E_CAPACITY;
  if (col_capacity > 0 && col_idx == nullptr) return SIFT_E_NULL;
  const bool bf16 = q->dtype == SIFT_BF16;
  if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale))
    softmax_scale = 1.0f / std::sqrt(static_cast<float>(in.head_dim));
  if ((st = check_device(plan)) != SIFT_OK) return st;
  sift::AttnArgs a{};
  a.q = q->data;
  a.k = k->data;
  a.v = v->data;
  a.out = out->data;
  a.row_ptr = row_ptr;
  a.col_idx = col_idx;
  a.col_capacity = col_capacity;
  a.hq = in.num_q_heads;
  a.hkv = in.num_kv_heads;
  a.head_dim = in.head_dim;
  a.tile = in.tile;
  a.scale_log2 = softmax_scale * 1.4426950408889634f;
  a.out_f32 = out->dtype == SIFT_F32 ? 1 : 0;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e;
  if (bf16) {
    // the bf16 kernel walks merged per-unit step lists: build them from the lists
    e = sift::launch_merge_steps(plan->pt, work(plan, false), row_ptr, col_idx, col_capacity, s);
    plan->steps_decoded = false;
    if (e == hipSuccess) plan->steps_paged = false;
    if (e == hipSuccess) e = sift::launch_attn_bf16(plan->pt, work(plan, false), a, s);
  } else {
    // the plan's steps stay the last decode's
    e = sift::launch_attn_f32(plan->pt, nullptr, a, s);
  }
  plan->last_stream = s;
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

// after_decode: the call's own decode precedes.
static sift_status attend(sift_plan* plan, const sift_tensor* q, const sift_tensor* k,
                          const sift_tensor* v, float softmax_scale, sift_tensor* out,
                          bool after_decode, bool sorted, void* stream) {
  if (plan == nullptr) return SIFT_E_NULL;
  const sift_plan_info& in = plan->info;
  sift_status st = check_io(q, k, v, out, in.num_tokens, in.num_q_heads, in.num_kv_heads,
                            in.head_dim, in.tile);
  if (st != SIFT_OK) return st;
  if (plan->steps_paged && q->dtype == SIFT_BF16) return SIFT_E_PLAN;  // steps index a page pool
  // fp32 inputs: over the steps where they are the last decode's, for packed K and V, or over
  // the plan's lists; neither is left when that decode wrote its lists to the caller's buffers
  // and attention over caller-given lists has replaced its steps (or there was no decode)
  const bool steps = plan->steps_decoded && !plan->steps_paged;
  if (q->dtype == SIFT_F32 && !plan->lists_own) {
    if (!steps) return SIFT_E_PLAN;
    if (!sift::f32_units_fit(plan->wt)) return SIFT_E_CAPACITY;  // steps that no launch could hold
  }
  if ((st = check_device(plan)) != SIFT_OK) return st;
  if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale))
    softmax_scale = 1.0f / std::sqrt(static_cast<float>(in.head_dim));
  sift::AttnArgs a{};
  a.q = q->data;
  a.k = k->data;
  a.v = v->data;
  a.out = out->data;
  a.row_ptr = plan->row_ptr;
  a.col_idx = plan->col_idx;
  a.col_capacity = in.list_capacity;
  a.hq = in.num_q_heads;
  a.hkv = in.num_kv_heads;
  a.head_dim = in.head_dim;
  a.tile = in.tile;
  a.scale_log2 = softmax_scale * 1.4426950408889634f;
  a.out_f32 = out->dtype == SIFT_F32 ? 1 : 0;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  if (!plan->lists_own) a.row_ptr = nullptr;  // never those of an older decode
  const sift::WorkTables wt = work(plan, sorted);
  hipError_t e;
  if (q->dtype == SIFT_BF16) {
    e = sift::launch_attn_bf16(plan->pt, wt, a, s);
  } else {
    // a graph that does not hold the decode replays over whatever the plan holds
    // then: its lists are a decode's, its steps may be page-pool rows or a bf16
    // call's merged lists
    const unsigned long long cap = after_decode ? 0 : capture_of(s);
    const bool keep = cap != 0 && cap != plan->decode_capture && plan->lists_own;
    e = sift::launch_attn_f32(plan->pt, steps && !keep ? &wt : nullptr, a, s);
  }
  plan->last_stream = s;
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

sift_status sift_plan_attention(sift_plan* plan, const sift_tensor* q, const sift_tensor* k,
                                const sift_tensor* v, float softmax_scale, sift_tensor* out,
                                void* stream) {
  return attend(plan, q, k, v, softmax_scale, out, false, false, stream);
}

sift_status sift_plan_run(sift_plan* plan, const sift_tensor* q, const sift_tensor* k,
                          const sift_tensor* v, const uint8_t* local_bitmap,
                          const uint8_t* cross_bitmap, float softmax_scale, sift_tensor* out,
                          void* stream) {
  if (plan == nullptr) return SIFT_E_NULL;
  const sift_plan_info& in = plan->info;
  // check everything before enqueuing the decode
  sift_status st = check_io(q, k, v, out, in.num_tokens, in.num_q_heads, in.num_kv_heads,
                            in.head_dim, in.tile);
  if (st != SIFT_OK) return st;
  if (in.la_bytes > 0 && local_bitmap == nullptr) return SIFT_E_NULL;
  if (in.ca_bytes > 0 && cross_bitmap == nullptr) return SIFT_E_NULL;
  const bool sorted = q->dtype == SIFT_F32;
  st = decode_lists(plan, local_bitmap, cross_bitmap, plan->row_ptr, plan->col_idx,
                    in.list_capacity, sorted, stream);
  if (st != SIFT_OK) return st;
  return attend(plan, q, k, v, softmax_scale, out, true, sorted, stream);
}


sift_status sift_plan_run_paged(sift_plan* plan, const sift_tensor* q, const sift_tensor* k_pages,
                                const sift_tensor* v_pages, const int32_t* page_table,
                                const uint8_t* local_bitmap, const uint8_t* cross_bitmap,
                                float softmax_scale, sift_tensor* out, void* stream) {
  if (plan == nullptr || k_pages == nullptr || v_pages == nullptr) return SIFT_E_NULL;
  const sift_plan_info& in = plan->info;
  sift_status st;
  if ((st = check_tensor(q, in.num_tokens, in.num_q_heads, in.head_dim)) != SIFT_OK) return st;
  if ((st = check_tensor(out, in.num_tokens, in.num_q_heads, in.head_dim)) != SIFT_OK) return st;
  // the pools: whole pages of T rows, at least one when there are tiles
  const int32_t rows = k_pages->tokens;
  if (rows < 0 || rows % in.tile != 0) return SIFT_E_SHAPE;
  const int32_t num_pages = rows / in.tile;
  if ((st = check_tensor(k_pages, rows, in.num_kv_heads, in.head_dim)) != SIFT_OK) return st;
  if ((st = check_tensor(v_pages, rows, in.num_kv_heads, in.head_dim)) != SIFT_OK) return st;
  if (in.num_tiles > 0 && num_pages < 1) return SIFT_E_SHAPE;
  if (in.num_tiles > 0 && page_table == nullptr) return SIFT_E_NULL;
  if (q->dtype != k_pages->dtype || q->dtype != v_pages->dtype) return SIFT_E_UNSUPPORTED;
  // bf16 at T < 64: a 64-key step's tiles each come from their own page
  if (q->dtype == SIFT_BF16 && in.head_dim != 128) return SIFT_E_UNSUPPORTED;
  if (q->dtype == SIFT_F32 && (out->dtype != SIFT_F32 || in.tile > 64)) return SIFT_E_UNSUPPORTED;
  if (in.la_bytes > 0 && local_bitmap == nullptr) return SIFT_E_NULL;
  if (in.ca_bytes > 0 && cross_bitmap == nullptr) return SIFT_E_NULL;
  if ((st = check_device(plan)) != SIFT_OK) return st;
  if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale))
    softmax_scale = 1.0f / std::sqrt(static_cast<float>(in.head_dim));
  const sift::KvPages pages{page_table, num_pages};
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const sift::WorkTables wt = work(plan, q->dtype == SIFT_F32);
  hipError_t e = sift::launch_decode(plan->pt, wt, local_bitmap, cross_bitmap, plan->counts,
                                     plan->row_ptr, plan->col_idx, pages, s);
  plan->last_stream = s;
  if (e != hipSuccess) return SIFT_E_HIP;
  plan->steps_paged = true;
  plan->steps_decoded = true;
  plan->lists_own = true;
  sift::AttnArgs a{};
  a.q = q->data;
  a.k = k_pages->data;
  a.v = v_pages->data;
  a.out = out->data;
  a.row_ptr = plan->row_ptr;
  a.col_idx = plan->col_idx;
  a.col_capacity = in.list_capacity;
  a.hq = in.num_q_heads;
  a.hkv = in.num_kv_heads;
  a.head_dim = in.head_dim;
  a.tile = in.tile;
  a.scale_log2 = softmax_scale * 1.4426950408889634f;
  a.out_f32 = out->dtype == SIFT_F32 ? 1 : 0;
  a.pages = pages;
  e = q->dtype == SIFT_BF16 ? sift::launch_attn_bf16(plan->pt, wt, a, s)
                            : sift::launch_attn_f32(plan->pt, &wt, a, s);
  plan->last_stream = s;
  return e == hipSuccess ? SIFT_OK : SIFT_E_HIP;
}

sift_status sift_sparse_prefill(const sift_tensor* q, const sift_tensor* k, const sift_tensor* v,
                                const sift_layout* doc_offsets, const uint8_t* local_bitmap,
                                const uint8_t* cross_bitmap, int32_t tile, sift_tensor* out,
                                void* stream) {
  PlanImage im;
  sift_status st = check_prefill(q, k, v, doc_offsets, local_bitmap, cross_bitmap, tile, out, im);
  if (st != SIFT_OK) return st;
  // stream-ordered scratch: allocated, used and freed in the order of `stream`
  const hipStream_t s = static_cast<hipStream_t>(stream);
  void* ws = nullptr;
  if (hipMallocAsync(&ws, im.total, s) != hipSuccess) return SIFT_E_HIP;
  sift_plan* plan = nullptr;
  st = create_plan(im, ws, im.total, s, Upload::kStaged, &plan);
  if (st == SIFT_OK)
    st = sift_plan_run(plan, q, k, v, local_bitmap, cross_bitmap, 0.f, out, stream);
  const sift_status st2 = sift_plan_destroy(plan);  // host state only: ws is freed below
  if (hipFreeAsync(ws, s) != hipSuccess && st == SIFT_OK) return SIFT_E_HIP;
  return st != SIFT_OK ? st : st2;
}

sift_status sift_sparse_prefill_ex(const sift_tensor* q, const sift_tensor* k,
                                   const sift_tensor* v, const sift_layout* doc_offsets,
                                   const uint8_t* local_bitmap, const uint8_t* cross_bitmap,
                                   int32_t tile, float softmax_scale, void* workspace,
                                   size_t workspace_bytes, sift_tensor* out, void* stream) {
  PlanImage im;
  sift_status st = check_prefill(q, k, v, doc_offsets, local_bitmap, cross_bitmap, tile, out, im);
  if (st != SIFT_OK) return st;
  if (workspace == nullptr) return SIFT_E_NULL;
  if (workspace_bytes < im.total) return SIFT_E_CAPACITY;
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return SIFT_E_UNSUPPORTED;
  sift_plan* plan = nullptr;
  st = create_plan(im, workspace, workspace_bytes, static_cast<hipStream_t>(stream),
                   Upload::kStaged, &plan);
  if (st != SIFT_OK) return st;
  st = sift_plan_run(plan, q, k, v, local_bitmap, cross_bitmap, softmax_scale, out, stream);
  const sift_status st2 = sift_plan_destroy(plan);  // host state only: the workspace is the caller's
  return st != SIFT_OK ? st : st2;
}

sift_status sift_decode_workspace_bytes(const sift_layout* layout, int32_t num_q_heads,
                                        int32_t tile, size_t* bytes) {
  return sift_workspace_bytes(layout, num_q_heads, kDecodeKvHeads, kDecodeHeadDim, tile, bytes);
}

sift_status sift_decode_tiles(const sift_layout* layout, const uint8_t* local_bitmap,
                              const uint8_t* cross_bitmap, int32_t tile, int32_t num_q_heads,
                              int32_t* row_ptr, int32_t* col_idx, int64_t col_capacity,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (layout == nullptr || row_ptr == nullptr || workspace == nullptr) return SIFT_E_NULL;
  if (num_q_heads < 1) return SIFT_E_SHAPE;
  if (tile != 16 && tile != 32 && tile != 64 && tile != 128) return SIFT_E_UNSUPPORTED;
  PlanImage im;
  sift_status st = make_image(layout, num_q_heads, kDecodeKvHeads, kDecodeHeadDim, tile, im);
  if (st != SIFT_OK) return st;
  const HostPlan& hp = im.hp;
  if (hp.la_bytes > 0 && local_bitmap == nullptr) return SIFT_E_NULL;
  if (hp.ca_bytes > 0 && cross_bitmap == nullptr) return SIFT_E_NULL;
  const int64_t cap = hp.dense_tiles * num_q_heads;
  if (cap > 0 && col_idx == nullptr) return SIFT_E_NULL;
  if (col_capacity < cap) return SIFT_E_CAPACITY;
  if (workspace_bytes < im.total) return SIFT_E_CAPACITY;
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return SIFT_E_UNSUPPORTED;
  sift_plan* plan = nullptr;
  st = create_plan(im, workspace, workspace_bytes, static_cast<hipStream_t>(stream),
                   Upload::kStaged, &plan);
  if (st != SIFT_OK) return st;
  st = sift_plan_decode_tiles(plan, local_bitmap, cross_bitmap, row_ptr, col_idx, col_capacity,
                              stream);
  const sift_status st2 = sift_plan_destroy(plan);  // host state only
  return st != SIFT_OK ? st : st2;
}

sift_status sift_sparse_prefill_static(const sift_tensor* q, const sift_tensor* k,
                                       const sift_tensor* v, const sift_layout* doc_offsets,
                                       const uint8_t* local_bitmap, const uint8_t* cross_bitmap,
                                       int32_t tile, float softmax_scale, sift_tensor* out,
                                       void* stream) {
  PlanImage im;
  sift_status st = check_prefill(q, k, v, doc_offsets, local_bitmap, cross_bitmap, tile, out, im);
  if (st != SIFT_OK) return st;
  if (im.total > kStaticScratchBytes) return SIFT_E_CAPACITY;
  void* ws = nullptr;
  if ((st = static_scratch(&ws)) != SIFT_OK) return st;
  // tables from host memory: the call waits for the copy, so nothing is
  // allocated to hold them
  sift_plan* plan = nullptr;
  st = create_plan(im, ws, kStaticScratchBytes, static_cast<hipStream_t>(stream),
                   Upload::kPageable, &plan);
  if (st != SIFT_OK) return st;
  st = sift_plan_run(plan, q, k, v, local_bitmap, cross_bitmap, softmax_scale, out, stream);
  const sift_status st2 = sift_plan_destroy(plan);  // host state only
  return st != SIFT_OK ? st : st2;
}

size_t sift_static_scratch_bytes(void) { return kStaticScratchBytes; }

}  // extern "C"
