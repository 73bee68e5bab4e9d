// C ABI of libbs_attn.so: argument validation, workspace layout, launch order.
// The declarations and the contract of every entry point are in bs_attn.h.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <vector>

#include "attn.hpp"

// Scratch of the allocation-free forward (bs_attn_varlen_fwd_noalloc): the plan that the
// forward kernel walks (header, per-segment offsets, work list), then the pieces of the
// few-query forward or the partials of split chains (kFewBytes).  Each device holds its own
// copy from the time the library's code is loaded on it until the process ends.  Host code
// never uses this name as an address: the device address comes from hipGetSymbolAddress.
constexpr size_t kNoAllocScratchBytes = BS_NOALLOC_SCRATCH_BYTES;
constexpr size_t kFewBytes = BS_NOALLOC_PIECE_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes + kFewBytes];

namespace bs {
namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

int ok() {
  g_err[0] = '\0';
  return BS_OK;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(BS_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr int64_t kMaxTokens = int64_t(1) << 30;
// query heads: keeps the byte offsets inside one tile of rows below 2^31
constexpr int32_t kMaxHeads = 4096;

// Profiling: pairs of HIP events recorded around each kernel launch while enabled.
struct Profiler {
  std::mutex mu;
  std::atomic<bool> on{false};
  std::vector<std::pair<hipEvent_t, hipEvent_t>> recs[BS_KERNEL_COUNT];
  std::vector<hipEvent_t> spare;
};

Profiler& prof() {
  static Profiler* p = new Profiler();  // never destroyed: events may outlive static teardown
  return *p;
}

hipEvent_t take_event() {
  Profiler& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  if (!P.spare.empty()) {
    hipEvent_t e = P.spare.back();
    P.spare.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

void give_back(hipEvent_t e) {
  if (e == nullptr) return;
  Profiler& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  P.spare.push_back(e);
}

// Records an event pair around the launches made during its lifetime (none when an event
// cannot be had: the one that was is returned to the pool).
class ProfScope {
 public:
  ProfScope(int kind, hipStream_t s) : kind_(kind), s_(s) {
    if (!prof().on.load(std::memory_order_relaxed)) return;
    a_ = take_event();
    b_ = take_event();
    if (a_ && b_) {
      hipEventRecord(a_, s_);
    } else {
      give_back(a_);
      give_back(b_);
      a_ = b_ = nullptr;
    }
  }
  ~ProfScope() {
    if (!a_ || !b_) return;
    hipEventRecord(b_, s_);
    Profiler& P = prof();
    std::lock_guard<std::mutex> g(P.mu);
    P.recs[kind_].emplace_back(a_, b_);
  }

 private:
  int kind_;
  hipStream_t s_;
  hipEvent_t a_ = nullptr, b_ = nullptr;
};

struct PlanCfg {
  PlanKind kind;
  int tile_a, tile_b;
};

bool is_bwd(int op) {
  return op == BS_OP_VARLEN_BWD || op == BS_OP_CHUNK_BWD || op == BS_OP_PACKED_CHUNK_BWD;
}
// ops whose problem is a list of segments (cu_seqlens)
bool is_varlen(int op) {
  return op == BS_OP_VARLEN_FWD || op == BS_OP_VARLEN_BWD || op == BS_OP_PACKED_CHUNK_FWD ||
         op == BS_OP_PACKED_CHUNK_BWD;
}
// segment ops whose diagonals come from per-segment global positions
bool is_packed(int op) { return op == BS_OP_PACKED_CHUNK_FWD || op == BS_OP_PACKED_CHUNK_BWD; }
// the backward that writes dQ itself (the others add into the caller's fp32 dq_accum)
bool writes_dq(int op) { return op == BS_OP_VARLEN_BWD; }
bool valid_op(int op) { return op >= BS_OP_VARLEN_FWD && op <= BS_OP_PACKED_CHUNK_BWD; }

// Plans an op runs, in launch order: the forward walks query tiles; the
// backward plans twice, query tiles for its dQ kernel, then key tiles for its
// dK/dV kernel.
int plans_of(int op, const bs_dims& d, PlanCfg out[2]) {
  if (d.dtype == BS_BF16) {
    out[0] = PlanCfg{kPlanFwd, kFwdBM, kFwdBN};
    out[1] = PlanCfg{kPlanBwd, kBwdBN, bwd_bm(d.head_dim)};
  } else {
    out[0] = PlanCfg{kPlanFwd, kF32BM, kF32BN};
    out[1] = PlanCfg{kPlanBwd, kF32BwdBN, kF32BwdBM};
  }
  return is_bwd(op) ? 2 : 1;
}

int64_t max_items_of(const PlanCfg& c, const bs_dims& d, int64_t nseg, bool varlen) {
  const int64_t ta = c.kind == kPlanFwd ? d.total_q : d.total_k;
  return (ta + c.tile_a - 1) / c.tile_a + (varlen ? nseg : 0);
}

int check_dims(const bs_dims* d, bool need_kv) {
  if (d == nullptr) return fail(BS_ERR_INVALID_ARG, "dims is NULL");
  if (d->dtype != BS_F32 && d->dtype != BS_BF16)
    return fail(BS_ERR_UNSUPPORTED, "dtype %d is not BS_F32 or BS_BF16", d->dtype);
  if (d->head_dim != 64 && d->head_dim != 128)
    return fail(BS_ERR_UNSUPPORTED, "head_dim %d is not 64 or 128", d->head_dim);
  if (d->hq < 1 || d->hq > kMaxHeads)
    return fail(BS_ERR_INVALID_ARG, "hq = %d out of [1, %d]", d->hq, kMaxHeads);
  if (d->total_q < 0 || d->total_q >= kMaxTokens)
    return fail(BS_ERR_INVALID_ARG, "total_q = %lld out of [0, 2^30)", (long long)d->total_q);
  if (need_kv) {
    if (d->hkv < 1 || d->hq % d->hkv != 0)
      return fail(BS_ERR_INVALID_ARG, "hq = %d must be a positive multiple of hkv = %d", d->hq, d->hkv);
    if (d->total_k < 0 || d->total_k >= kMaxTokens)
      return fail(BS_ERR_INVALID_ARG, "total_k = %lld out of [0, 2^30)", (long long)d->total_k);
  }
  return BS_OK;
}

int check_ptr(const void* p, int64_t count, const char* name) {
  if (count == 0) return BS_OK;
  if (p == nullptr) return fail(BS_ERR_INVALID_ARG, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(p) % 16 != 0)
    return fail(BS_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
  return BS_OK;
}

int check_scale(float s) {
  if (!isfinite(s) || !(s > 0.f)) return fail(BS_ERR_INVALID_ARG, "scale must be finite and > 0");
  return BS_OK;
}

// How a bf16 kernel of few workgroups runs: by its own plan (no list), each work item's chain of
// tiles split over `splits` workgroups.
struct SelfCfg {
  bool self;
  int32_t splits;
  int64_t items, wgs;
  size_t bytes;  // of the partials (0: none)
  double us;     // the estimate below
};
enum SelfKernel { kSelfFwd, kSelfDq, kSelfDkdv };

// The rule, from the sizes: at most as many workgroups as the chip holds at once (two per CU for
// the forward and dQ, one for dK/dV), or less than half as many again where no segment is longer
// than 512; and the number of parts (at most 8) with the smallest estimate in microseconds
//   rounds of workgroups x chain / parts x t  +  (with parts) 5 for the second kernel and the
//   partials' bytes, written and read, at 3 TB/s,
// t = 0.65 per 64-key tile (forward), 0.9 (dQ), 1.9 per 96-row step (dK/dV; 1.2 per 64-row one;
// float32: 7.5 per 128-row step, 3.8 at head_dim 64), the measured times of a chain on a CU.
// Forward + backward, us, by the list / so:
//   512 tokens, 8/8 heads: 55 / 49    505, 64/8: 99 / 68    628, 32/4: 134 / 70    864, 32/32: 61 / 56
// and a 1,018-token ring of three steps, 8/8 heads: 415 / 347 to 388; a 4-way zig-zag share of 1,240,
// 480 and 2,000 tokens, 16/2 heads: 896 / 505 (head_dim 64: 692 / 382).  Beyond the lines the gain
// falls off (2,671 tokens, 32/32, 832 workgroups: 164 / 165; 1,875, 40/8, 800 workgroups: 171 / 168; 2,413, 32/32, 800: 184 / 176).
// Partials: 16 MiB at most in the forward (what the allocation-free entry point holds), 64 MiB in
// the backward.
constexpr int64_t kSelfShort = 512;

// The longest segment that the estimates count on: max_seqlen is only a bound (a context's or a
// buffer's length, say), so at most four times the mean.  With the bound itself, 2,660 tokens in 32
// segments of up to 139, 4/1 heads, max_seqlen 2,660, forward: 55 us (four parts of chains of two
// tiles); so 11.
int64_t likely_longest(int64_t bound, int64_t total, int64_t nseg) {
  const int64_t four = nseg > 4 ? 4 * ((total + nseg - 1) / nseg) : total;
  return bound < four ? bound : four;
}
// seen: queries or keys that the longest chain walks at most, where that is known.
SelfCfg self_cfg(SelfKernel k, int op, const bs_dims& d, int64_t nseg, int64_t max_seqlen,
                 int64_t seen = INT64_MAX) {
  SelfCfg c = {false, 1, 0, 0, 0, 0};
  const bool varlen = is_varlen(op);
  const bool f32 = d.dtype == BS_F32;  // dK/dV's chains alone are split there, by the list
  if ((f32 && k != kSelfDkdv) || (varlen && (nseg < 1 || (!f32 && nseg > kSelfMaxSegs)))) return c;
  PlanCfg cfg[2];
  plans_of(op, d, cfg);
  const bool dkdv = k == kSelfDkdv;
  const int64_t slots = dkdv ? 256 : 512;
  c.items = max_items_of(cfg[dkdv ? 1 : 0], d, nseg, varlen);
  const int64_t wgs = c.wgs = c.items * (dkdv ? d.hkv : d.hq);
  const int64_t len = dkdv ? d.total_q : d.total_k;
  const int64_t longest = varlen && max_seqlen < len ? max_seqlen : len;
  const bool more = !f32 && longest <= kSelfShort;
  if (wgs < 1 || (more ? 2 * wgs >= 3 * slots : wgs > slots)) return c;
  c.self = !f32;
  const int64_t likely = likely_longest(longest, len, varlen ? nseg : 1);
  const int64_t bm = f32 ? kF32BwdBM : bwd_bm(d.head_dim), walk = likely < seen ? likely : seen;
  const double chain = dkdv ? (double)((walk + bm - 1) / bm * (d.hq / d.hkv)) : walk / 64.0;
  const double t = f32 ? (d.head_dim == 128 ? 7.5 : 3.8)
                 : dkdv ? (d.head_dim == 128 ? 1.9 : 1.2) : (k == kSelfFwd ? 0.65 : 0.9);
  const size_t rows = dkdv ? (size_t)(2 * d.total_k * d.hkv) : (size_t)(d.total_q * d.hq);
  const size_t slab = rows * (d.head_dim + (k == kSelfFwd ? 2 : 0)) * sizeof(float);
  if (rows == 0) return c;  // no output rows (all segments lack queries, or keys): nothing to share
  const size_t limit = k == kSelfFwd ? kFewBytes : (size_t)64 << 20;
  for (int32_t s = 1; s <= 8 && s <= chain && (s == 1 || s * slab <= limit); ++s) {
    const double cost = (double)((wgs * s + slots - 1) / slots) * chain / s * t +
                        (s > 1 ? 5 + 2e-6 * (double)(s * slab) / 3 : 0);
    if (s == 1 || cost < c.us) {
      c.us = cost;
      c.splits = s;
    }
  }
  c.bytes = c.splits > 1 ? align256(c.splits * slab) : 0;
  return c;
}

// The form of one call.  A causal chunk's offsets tell how long its chains are at most, and so
// whether sharing them pays (they do not change which form the sizes ask for, nor its room).  A
// 326-query chunk whose keys of 5,463 it sees the first 326 of, 32/4 heads, forward: in 4 parts 24 us,
// unsplit 11.
SelfCfg self_cfg_at(SelfKernel k, int op, const bs_dims& d, int64_t nseg, int64_t max_seqlen,
                    int64_t q_off, int64_t k_off, int causal) {
  SelfCfg c = self_cfg(k, op, d, nseg, max_seqlen);
  if (c.splits == 1 || is_varlen(op) || !causal) return c;
  // key j visible to query i iff j <= i + diag: query tiles see total_q + diag keys at most, key
  // tiles are seen from query -diag on
  int64_t diag = q_off - k_off;
  diag = diag < -kDiagClamp ? -kDiagClamp : (diag > kDiagClamp ? kDiagClamp : diag);
  const int64_t seen = k != kSelfDkdv ? d.total_q + diag : (diag < 0 ? d.total_q + diag : d.total_q);
  const int32_t splits = self_cfg(k, op, d, nseg, max_seqlen, seen > 0 ? seen : 0).splits;
  if (splits < c.splits) c.splits = splits;
  return c;
}

// Whether a varlen forward takes the few-query kernel, from the sizes alone, and its buffers.
//
// The rule compares two estimates in microseconds (segments taken as equally long), a pair of them for
// each form that the general path would take, fitted to calls of MHA and GQA, training, prompts and
// decoding, over up to 16K keys (self-planned: 1,400 of 1..64 segments, checked on 953 more of 1..256;
// by the list: 2,000 of 1..1,024):
//   self-planned: 6, 0.06 per segment and 1 per 128 workgroups beyond 256 (3.2 of these alone for
//     segments as stored), and the larger of 0.9 of that form's own estimate and the key bytes at
//     3.9 TB/s; 9.7 at least (below it the two are 1 to 3 us apart, and the smallest calls stay
//     with few queries);
//   few-query against it: 4, +5 for the merge, 4 per row block that a workgroup starts on average,
//     and the larger of the key bytes at 5.3 TB/s (a third of that again for each further row block
//     that reads them) and 1.6 per 128 keys of a 32-row block, shared evenly by 512 workgroups
//     unless the bound on a row's pieces leaves some of them idle;
//   by the list: 9.9, 0.13 per segment, and the larger of the key bytes at 5.6 TB/s and 2.6 + 1.28 per
//     64-key tile for each round of 512 workgroups (one per 128-row tile of a head);
//   few-query against it: 6.1, +4.6 for the merge, 2 and up to 1.7 more, by how full it is, for each
//     row block that a workgroup starts, and the key bytes at 7 TB/s with 0.65 of that again for each
//     further row block that reads them, longer where workgroups are idle.
// The choice is on average 3.8 % and 0.2 % above the better of the two.  Measured on both sides, us
// (few / general; segments x queries, longest segment, heads; head_dim 128):
//   32x1 8K 64/8: 78 / 355    16x8 4K 32/32: 94 / 126    1x1 16K 64/8: 26 / 70
//   4x1 1K 32/8: 12 / 14      70x1 139 12/2: 11 / 24     70x1 139 7/7: 14 / 15
//   4x32 4K 64/8: 65 / 58     2x128 8K 32/32: 141 / 53   1x170 170 40/8: 15 / 9
//   2 segments of 452 and 60, 8/8: 17 / 13   of 114 and 294, 16/16: 18 / 11   1x8 160 48/8: 11 / 7
//   199x63 104 32/8: 145 / 112   114x1 79 64/64: 69 / 84   39x23 2.2K 16/16: 137 / 100
// and calls whose queries x heads leave room for fewer than two pieces per row (16 MiB, over
// about 16K rows) stay on the general path.
// per_min: key blocks per workgroup at least, as expected.
bool few_pays(const bs_dims& d, int64_t nseq, const FewLayout& F, int32_t per_min, const SelfCfg& self) {
  const double n = (double)nseq, group = (double)d.hq / d.hkv, lq = d.total_q / n, lk = d.total_k / n;
  const double mb = (double)d.total_k * d.hkv * d.head_dim * 4e-6;
  if (self.self) {
    const double rows = d.total_q * group, keys = lk / 128 + 1;
    const double rb = rows / 32 + nseq / 2 > n ? rows / 32 + nseq / 2 : n;
    const double per_wg = rb * d.hkv / 512, blocks = per_wg * keys * 128 / few_block_keys(d.head_dim);
    const double few_c = 1.6 * keys * per_wg, few_m = mb / 5.3 * (1 + 0.35 * (rb / n - 1));
    const double few = 4 + (F.slabs > 1 ? 5 : 0) + 4 * per_wg +
                       (few_c > few_m ? few_c : few_m) * (per_min > blocks && blocks > 1 ? per_min / blocks : 1);
    const double gen_c = 0.9 * self.us, gen_m = mb / 3.9;
    const double over = self.wgs > 256 ? (self.wgs - 256) / 128.0 : 0;
    const double gen = 6 + (nseq <= kSelfRankSegs ? 0.06 * n + over : 3.2 * over) + (gen_c > gen_m ? gen_c : gen_m);
    return few < (gen > 9.7 ? gen : 9.7);
  }
  // tiles of a segment of on average x tiles: half a tile is lost, and no segment has less than one
  auto whole = [](double x) { return x > 0.5 ? x + 0.5 : 1; };
  // row blocks of a segment (a few queries on average are often one for most and many for some)
  const double spread = 1 + 0.8 * (lq - 1) * group / 32, even = whole(lq * group / 32);
  const double rb = even > spread ? even : spread, kb = whole(lk / few_block_keys(d.head_dim));
  const double blocks = n * rb * kb * d.hkv / 512, least = blocks > 1 ? blocks : 1;
  double per = ceil(blocks - 0.2);  // key blocks of a workgroup
  if (per < per_min) per = per_min;
  const double starts = per > kb ? per / kb : 1, full = lq * group / rb / 32;
  const double few = 6.1 + (F.slabs > 1 ? 4.6 : 0) + starts * (2 + 1.7 * (full < 1 ? full : 1)) +
                     mb / 7 * (1 + 0.65 * (rb - 1)) * (per_min > least ? per_min / least : 1);
  const double rounds = n * whole(lq / 128) * d.hq / 512;
  const double gen_c = (rounds > 1 ? rounds : 1) * (2.6 + 1.28 * (lk / 64 + 0.5)), gen_m = mb / 5.6;
  return few < 9.9 + 0.13 * n + (gen_c > gen_m ? gen_c : gen_m);
}

FewLayout few_layout(int op, const bs_dims& d, int64_t nseq, int64_t max_seqlen) {
  FewLayout F = {};
  if (op != BS_OP_VARLEN_FWD || d.dtype != BS_BF16 || nseq < 1 || nseq > kFewMaxSegs) return F;
  if (d.total_q < 1 || d.total_k < 1) return F;
  const int64_t group = d.hq / d.hkv, rows = d.total_q * d.hq, blk = few_block_keys(d.head_dim);
  // the line of key blocks: row blocks x key blocks of every segment, 32-bit per KV head
  const int64_t line = (d.total_q * group / 32 + nseq) * (d.total_k / blk + nseq);
  if (line >= (int64_t(1) << 31)) return F;
  const int64_t longest = max_seqlen < d.total_k ? max_seqlen : d.total_k;
  const int64_t likely = likely_longest(longest, d.total_k, nseq);
  int32_t per_likely = 1;
  if (longest <= blk) {  // one key block per segment at most
    F.slabs = F.per_min = 1;
    F.bytes = 256;
  } else {
    const size_t row_bytes = (size_t)(d.head_dim + 2) * sizeof(float);
    F.stat = align256(sizeof(int32_t) * (size_t)rows);
    if (F.stat + 512 + 2 * (size_t)rows * row_bytes > kFewBytes) return FewLayout{};
    const size_t fit = (kFewBytes - F.stat - 512) / ((size_t)rows * row_bytes);
    F.slabs = fit < kFewSlabs ? (int32_t)fit : kFewSlabs;
    F.per_min = few_per_min((int32_t)((longest + blk - 1) / blk), F.slabs);
    per_likely = few_per_min((int32_t)((likely + blk - 1) / blk), F.slabs);
    F.part = F.stat + align256(sizeof(float) * 2 * (size_t)(rows * F.slabs));
    F.bytes = F.part + align256(sizeof(float) * (size_t)(rows * F.slabs * d.head_dim));
  }
  if (!few_pays(d, nseq, F, per_likely, self_cfg(kSelfFwd, op, d, nseq, max_seqlen))) return FewLayout{};
  const int64_t wgs = line * d.hkv;
  F.blocks = wgs < 512 ? (int32_t)wgs : 512;  // two per CU
  return F;
}

// Room beyond the plan and D.  A float32 backward asks for at least what the bf16 call of its
// sizes does, so that its workspace also holds that call.
size_t extra_bytes(int op, bs_dims d, int64_t nseg, int64_t max_seqlen) {
  if (is_bwd(op) && d.dtype == BS_F32) {
    const size_t own = self_cfg(kSelfDkdv, op, d, nseg, max_seqlen).bytes;
    d.dtype = BS_BF16;
    const size_t as_bf16 = extra_bytes(op, d, nseg, max_seqlen);
    return own > as_bf16 ? own : as_bf16;
  }
  if (!is_bwd(op)) {
    const size_t a = few_layout(op, d, nseg, max_seqlen).bytes;
    return a != 0 ? a : self_cfg(kSelfFwd, op, d, nseg, max_seqlen).bytes;
  }
  const SelfCfg a = self_cfg(kSelfDq, op, d, nseg, max_seqlen);
  const SelfCfg b = self_cfg(kSelfDkdv, op, d, nseg, max_seqlen);
  if (!a.self && !b.self && nseg <= kPlanFusedSegs) {  // the second list of one planning launch
    PlanCfg cfg[2];
    plans_of(op, d, cfg);
    const int64_t items = max_items_of(cfg[1], d, nseg, is_varlen(op));
    return sizeof(WsHeader) + align256(sizeof(WorkItem) * (size_t)items);
  }
  return a.bytes > b.bytes ? a.bytes : b.bytes;
}

WsLayout layout_of(int op, const bs_dims& d, int64_t nseg, int64_t max_seqlen) {
  WsLayout L = {};
  PlanCfg cfg[2];
  const int np = plans_of(op, d, cfg);
  const bool varlen = is_varlen(op);
  int64_t mi = 0;
  for (int i = 0; i < np; ++i) {
    const int64_t m = max_items_of(cfg[i], d, nseg, varlen);
    mi = m > mi ? m : mi;
  }
  size_t off = align256(sizeof(WsHeader));
  L.seg_off = off;
  off += align256(sizeof(int32_t) * (size_t)(nseg + 2));
  L.seg_dst = off;
  off += align256(sizeof(int32_t) * (size_t)(nseg + 1));
  L.sorted = off;
  off += align256(sizeof(WorkItem) * (size_t)mi);
  if (is_bwd(op)) {
    L.dvec = off;
    off += align256(sizeof(float) * (size_t)(d.hq * d.total_q));
    if (writes_dq(op) && d.dtype == BS_F32) {  // (bwd_common says when it is used)
      L.dq_late = off;
      off += align256(sizeof(float) * (size_t)(d.total_q * d.hq * d.head_dim));
    }
  }
  L.extra = off;
  L.total = off + extra_bytes(op, d, nseg, max_seqlen);
  L.max_items = mi;
  return L;
}

int check_ws(const WsLayout& L, const void* ws, size_t bytes) {
  if (ws == nullptr) return fail(BS_ERR_WORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) % 256 != 0)
    return fail(BS_ERR_WORKSPACE, "workspace is not 256-byte aligned");
  if (bytes < L.extra)  // without the rest no chain is split, nor the few-query forward taken
    return fail(BS_ERR_WORKSPACE, "workspace of %zu bytes is smaller than the %zu required", bytes,
                L.total);
  return BS_OK;
}

// Runs plan `i` of the op; returns the layout with max_items set for that plan.
hipError_t run_plan(int op, const bs_dims& d, int i, const int32_t* cu_q, const int32_t* cu_k,
                    const int64_t* q_pos, const int64_t* k_pos, int32_t num_seqs,
                    int32_t max_seqlen, int64_t q_off, int64_t k_off, int causal, void* ws,
                    const WsLayout& L, WsLayout* Lp, hipStream_t s, const PlanSecond* second = nullptr) {
  PlanCfg cfg[2];
  plans_of(op, d, cfg);
  const bool varlen = is_varlen(op);
  *Lp = L;
  Lp->max_items = max_items_of(cfg[i], d, varlen ? num_seqs : 1, varlen);
  int64_t diag = q_off - k_off;
  diag = diag < -kDiagClamp ? -kDiagClamp : (diag > kDiagClamp ? kDiagClamp : diag);
  const bool packed = is_packed(op);
  return launch_plan(cfg[i].kind, varlen ? cu_q : nullptr, varlen ? cu_k : nullptr,
                     packed ? q_pos : nullptr, packed ? k_pos : nullptr,
                     varlen ? num_seqs : 1, d.total_q, d.total_k, max_seqlen, (int32_t)diag,
                     causal, cfg[i].tile_a, cfg[i].tile_b, Lp->max_items, ws, *Lp, second, s);
}

// The self-planned form of a kernel for this call (NULL: by the list); buf: room for partials
// or NULL.
const SelfPlan* self_plan_of(SelfKernel k, int op, const bs_dims& d, const int32_t* cu_q,
                             const int32_t* cu_k, const int64_t* q_pos, const int64_t* k_pos,
                             int32_t num_seqs, int32_t max_seqlen, int64_t q_off, int64_t k_off,
                             int causal, void* ws, void* buf, SelfPlan* sp) {
  const SelfCfg c = self_cfg_at(k, op, d, is_varlen(op) ? num_seqs : 1, max_seqlen, q_off, k_off, causal);
  if (!c.self) return nullptr;
  const int64_t diag = q_off - k_off;
  PlanArgs& a = sp->plan;
  a.cu_q = is_varlen(op) ? cu_q : nullptr;
  a.cu_k = is_varlen(op) ? cu_k : nullptr;
  a.q_pos = is_packed(op) ? q_pos : nullptr;
  a.k_pos = is_packed(op) ? k_pos : nullptr;
  a.hdr = static_cast<WsHeader*>(ws);
  a.total_q = d.total_q;
  a.total_k = d.total_k;
  a.num_seqs = num_seqs;
  a.max_seqlen = max_seqlen;
  a.diag_chunk = (int32_t)(diag < -kDiagClamp ? -kDiagClamp : (diag > kDiagClamp ? kDiagClamp : diag));
  sp->items = c.items;
  sp->splits = buf != nullptr ? c.splits : 1;
  sp->part = static_cast<float*>(buf);
  return sp;
}

int check_varlen_args(int op, const int32_t* cu_q, const int32_t* cu_k, const int64_t* q_pos,
                      const int64_t* k_pos, int32_t num_seqs, int32_t max_seqlen) {
  if (num_seqs < 0) return fail(BS_ERR_INVALID_ARG, "num_seqs = %d < 0", num_seqs);
  if (max_seqlen < 0) return fail(BS_ERR_INVALID_ARG, "max_seqlen = %d < 0", max_seqlen);
  if (cu_q == nullptr || cu_k == nullptr) return fail(BS_ERR_INVALID_ARG, "cu_seqlens is NULL");
  if (is_packed(op) && num_seqs > 0 && (q_pos == nullptr || k_pos == nullptr))
    return fail(BS_ERR_INVALID_ARG, "q_pos / k_pos is NULL");
  return BS_OK;
}

#define BS_TRY(x)                 \
  do {                            \
    int rc__ = (x);               \
    if (rc__ != BS_OK) return rc__; \
  } while (0)
#define BS_HIP(x, what)                        \
  do {                                         \
    hipError_t e__ = (x);                      \
    if (e__ != hipSuccess) return hip_fail(e__, what); \
  } while (0)

// True when the byte ranges [a, a + na) and [b, b + nb) intersect.
bool overlaps(const void* a, int64_t na, const void* b, int64_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return na > 0 && nb > 0 && x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

// merge == NULL: writes the step's (out, lse).  Otherwise folds the step into the
// running (merge->o_run, merge->lse_run); out is then optional (the final output).  pieces:
// kFewBytes for the few-query forward, or NULL: what the workspace holds beyond the plan.
int fwd_common(int op, const bs_dims* dims, const void* q, const void* k, const void* v,
               const int32_t* cu_q, const int32_t* cu_k, const int64_t* q_pos,
               const int64_t* k_pos, int32_t num_seqs, int32_t max_seqlen, int64_t q_off,
               int64_t k_off, int causal, float scale, void* out, float* lse,
               const FwdMerge* merge, void* ws, size_t ws_bytes, void* pieces, void* stream) {
  BS_TRY(check_dims(dims, true));
  const bs_dims& d = *dims;
  const int64_t qn = d.total_q * d.hq * d.head_dim, kn = d.total_k * d.hkv * d.head_dim;
  BS_TRY(check_ptr(q, qn, "q"));
  BS_TRY(check_ptr(k, kn, "k"));
  BS_TRY(check_ptr(v, kn, "v"));
  if (merge == nullptr) {
    BS_TRY(check_ptr(out, qn, "out"));
    BS_TRY(check_ptr(lse, d.total_q * d.hq, "lse"));
  } else {
    BS_TRY(check_ptr(merge->o_run, qn, "o_run"));
    BS_TRY(check_ptr(merge->lse_run, d.total_q * d.hq, "lse_run"));
    if (out != nullptr) {
      BS_TRY(check_ptr(out, qn, "out"));
      if (overlaps(out, qn * (d.dtype == BS_BF16 ? 2 : 4), merge->o_run, qn * 4))
        return fail(BS_ERR_INVALID_ARG, "out overlaps o_run");
    }
  }
  BS_TRY(check_scale(scale));
  if (is_varlen(op)) BS_TRY(check_varlen_args(op, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen));
  const WsLayout L = layout_of(op, d, is_varlen(op) ? num_seqs : 1, max_seqlen);
  BS_TRY(check_ws(L, ws, ws_bytes));
  hipStream_t s = static_cast<hipStream_t>(stream);
  const FewLayout F = few_layout(op, d, num_seqs, max_seqlen);
  if (F.bytes != 0 && (pieces != nullptr || ws_bytes >= L.total)) {
    ProfScope ps(BS_KERNEL_FWD, s);
    BS_HIP(launch_few_fwd(d, q, k, v, cu_q, cu_k, num_seqs, max_seqlen, causal, scale, out, lse, ws,
                          pieces != nullptr ? pieces : static_cast<char*>(ws) + L.extra, F, s),
           "few-query forward launch");
    return ok();
  }
  WsLayout Lp = L;
  SelfPlan sp;
  void* buf = pieces != nullptr ? pieces : (ws_bytes >= L.total ? static_cast<char*>(ws) + L.extra : nullptr);
  const SelfPlan* self = self_plan_of(kSelfFwd, op, d, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen,
                                      q_off, k_off, causal, ws, buf, &sp);
  if (self == nullptr) {
    ProfScope ps(BS_KERNEL_PLAN, s);
    BS_HIP(run_plan(op, d, 0, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen, q_off, k_off,
                    causal, ws, L, &Lp, s),
           "planner launch");
  }
  ProfScope ps(BS_KERNEL_FWD, s);
  if (d.dtype == BS_BF16) {
    BS_HIP(launch_fwd_bf16(d, q, k, v, causal, scale, out, lse, merge, ws, Lp, self, s),
           "forward launch");
    if (self != nullptr && self->splits > 1)
      BS_HIP(launch_fwd_combine(d, *self, out, lse, merge, s), "forward combine launch");
  } else
    BS_HIP(launch_fwd_f32(d, q, k, v, causal, scale, out, lse, merge, ws, Lp, s),
           "forward launch");
  return ok();
}

int bwd_common(int op, const bs_dims* dims, const void* q, const void* k, const void* v,
               const void* out, const float* lse, const void* dout, const int32_t* cu_q,
               const int32_t* cu_k, const int64_t* q_pos, const int64_t* k_pos,
               int32_t num_seqs, int32_t max_seqlen, int64_t q_off, int64_t k_off, int causal,
               float scale, float* dq_accum, void* dq, void* dk, void* dv, int kv_accumulate,
               void* ws, size_t ws_bytes, void* stream) {
  BS_TRY(check_dims(dims, true));
  const bs_dims& d = *dims;
  const int64_t qn = d.total_q * d.hq * d.head_dim, kn = d.total_k * d.hkv * d.head_dim;
  BS_TRY(check_ptr(q, qn, "q"));
  BS_TRY(check_ptr(k, kn, "k"));
  BS_TRY(check_ptr(v, kn, "v"));
  BS_TRY(check_ptr(out, qn, "out"));
  BS_TRY(check_ptr(lse, d.total_q * d.hq, "lse"));
  BS_TRY(check_ptr(dout, qn, "dout"));
  BS_TRY(check_ptr(dk, kn, "dk"));
  BS_TRY(check_ptr(dv, kn, "dv"));
  const bool varlen = is_varlen(op), direct = writes_dq(op);
  if (direct) BS_TRY(check_ptr(dq, qn, "dq"));
  else BS_TRY(check_ptr(dq_accum, qn, "dq_accum"));
  BS_TRY(check_scale(scale));
  if (varlen) BS_TRY(check_varlen_args(op, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen));
  const WsLayout L = layout_of(op, d, varlen ? num_seqs : 1, max_seqlen);
  BS_TRY(check_ws(L, ws, ws_bytes));
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  float* dvec = reinterpret_cast<float*>(base + L.dvec);
  const bool f32 = d.dtype == BS_F32;
  // A float32 varlen dq may take the place of an input (dq == q, a reused buffer): the kernels that
  // follow the dQ kernel still read that, so dq is written last, from the workspace.
  auto over = [&](const void* x, int64_t n) { return overlaps(dq, qn * 4, x, n * 4); };
  const bool late = f32 && direct && (over(q, qn) || over(k, kn) || over(v, kn) || over(out, qn) ||
                                      over(dout, qn) || over(lse, d.total_q * d.hq));
  float* dq_late = reinterpret_cast<float*>(base + L.dq_late);
  void* dq_to = late ? dq_late : (direct ? dq : dq_accum);
  WsLayout Lp = L;
  SelfPlan sp;
  void* buf = ws_bytes >= L.total ? base + L.extra : nullptr;
  const SelfPlan* self = self_plan_of(kSelfDq, op, d, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen,
                                      q_off, k_off, causal, ws, buf, &sp);
  const WsHeader* hdr = static_cast<const WsHeader*>(ws);
  // both lists by one launch where neither kernel plans for itself and there is room for two
  PlanCfg cfg[2];
  plans_of(op, d, cfg);
  const int64_t nseg = varlen ? num_seqs : 1;
  PlanSecond second = {cfg[1].kind, cfg[1].tile_a, cfg[1].tile_b, max_items_of(cfg[1], d, nseg, varlen), buf};
  const bool both = !f32 && buf != nullptr && nseg <= kPlanFusedSegs &&
                    !self_cfg(kSelfDq, op, d, nseg, max_seqlen).self &&
                    !self_cfg(kSelfDkdv, op, d, nseg, max_seqlen).self;
  if (self == nullptr) {
    ProfScope ps(BS_KERNEL_PLAN, s);
    BS_HIP(run_plan(op, d, 0, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen, q_off, k_off,
                    causal, ws, L, &Lp, s, both ? &second : nullptr),
           "planner launch");
  }
  {
    ProfScope ps(BS_KERNEL_BWD_DQ, s);
    if (f32)
      BS_HIP(launch_dq_f32(d, q, k, v, out, dout, lse, dvec, causal, scale, dq_to, !direct, ws, Lp, s),
             "backward dQ launch");
    else
      BS_HIP(launch_dq_bf16(d, q, k, v, out, dout, lse, dvec, causal, scale, direct ? dq : nullptr,
                            dq_accum, ws, Lp, self, s),
             "backward dQ launch");
    if (self != nullptr && self->splits > 1)
      BS_HIP(launch_sum_slabs(self->part, self->splits, qn, direct ? dq : dq_accum, nullptr,
                              direct ? kSumBf16 : kSumAddF32, hdr, s),
             "dQ sum launch");
  }
  self = self_plan_of(kSelfDkdv, op, d, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen, q_off, k_off,
                      causal, ws, buf, &sp);
  Lp = L;
  const void* list = ws;
  if (both) {
    list = buf;
    Lp.sorted = sizeof(WsHeader);
    Lp.max_items = second.max_items;
  } else if (self == nullptr) {
    ProfScope ps(BS_KERNEL_PLAN, s);
    BS_HIP(run_plan(op, d, 1, cu_q, cu_k, q_pos, k_pos, num_seqs, max_seqlen, q_off, k_off,
                    causal, ws, L, &Lp, s),
           "planner launch");
  }
  {
    ProfScope ps(BS_KERNEL_BWD_DKDV, s);
    if (f32) {
      const SelfCfg c = self_cfg_at(kSelfDkdv, op, d, nseg, max_seqlen, q_off, k_off, causal);
      const int32_t splits = buf != nullptr ? c.splits : 1;
      float* part = static_cast<float*>(buf);
      BS_HIP(launch_dkdv_f32(d, q, k, v, dout, lse, dvec, causal, scale, dk, dv, kv_accumulate, ws,
                             Lp, splits, part, s),
             "backward dK/dV launch");
      if (splits > 1)
        BS_HIP(launch_sum_slabs(part, splits, kn, dk, dv, kv_accumulate ? kSumAddF32 : kSumF32, hdr, s),
               "dK/dV sum launch");
    } else {
      BS_HIP(launch_dkdv_bf16(d, q, k, v, dout, lse, dvec, causal, scale, dk, dv, kv_accumulate,
                              list, Lp, self, s),
             "backward dK/dV launch");
      if (self != nullptr && self->splits > 1)
        BS_HIP(launch_sum_slabs(self->part, self->splits, kn, dk, dv,
                                kv_accumulate ? kSumAddF32 : kSumBf16, hdr, s),
               "dK/dV sum launch");
    }
  }
  if (late) {
    ProfScope ps(BS_KERNEL_FINALIZE, s);
    BS_HIP(launch_sum_slabs(dq_late, 1, qn, dq, nullptr, kSumF32, hdr, s), "dQ copy launch");
  }
  return ok();
}

// Device address of `scratch` on each device, looked up once per device (with that device
// current) on the first allocation-free call made there.
constexpr int kMaxScratchDevices = 256;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxScratchDevices] = {};

int noalloc_scratch(void* stream, void** addr) {
  int dev = -1;
  BS_HIP(hipGetDevice(&dev), "hipGetDevice");
  if (stream != nullptr) {
    int sdev = -1;
    BS_HIP(hipStreamGetDevice(static_cast<hipStream_t>(stream), &sdev), "hipStreamGetDevice");
    if (sdev != dev)
      return fail(BS_ERR_INVALID_ARG, "stream belongs to device %d but device %d is current", sdev,
                  dev);
  }
  if (dev < 0 || dev >= kMaxScratchDevices)
    return fail(BS_ERR_UNSUPPORTED, "device %d is beyond the %d devices with scratch slots", dev,
                kMaxScratchDevices);
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (g_scratch_addr[dev] == nullptr) {
    void* p = nullptr;
    BS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (p == nullptr) return fail(BS_ERR_HIP, "hipGetSymbolAddress(scratch) returned NULL");
    g_scratch_addr[dev] = p;
  }
  *addr = g_scratch_addr[dev];
  return BS_OK;
}

}  // namespace
}  // namespace bs

using namespace bs;

extern "C" {

size_t bs_attn_workspace_size(int op, const bs_dims* dims, int32_t num_seqs, int32_t max_seqlen) {
  if (!valid_op(op)) {
    fail(BS_ERR_UNSUPPORTED, "unknown op %d", op);
    return 0;
  }
  if (check_dims(dims, true) != BS_OK) return 0;
  if (is_varlen(op) && (num_seqs < 0 || max_seqlen < 0)) {
    fail(BS_ERR_INVALID_ARG, "num_seqs and max_seqlen must be >= 0");
    return 0;
  }
  ok();
  return layout_of(op, *dims, is_varlen(op) ? num_seqs : 1, max_seqlen).total;
}

int bs_attn_varlen_fwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                       const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k, int32_t num_seqs,
                       int32_t max_seqlen, int causal, float scale, void* out, float* lse,
                       void* workspace, size_t workspace_bytes, void* stream) {
  return fwd_common(BS_OP_VARLEN_FWD, dims, q, k, v, cu_seqlens_q, cu_seqlens_k, nullptr, nullptr,
                    num_seqs, max_seqlen, 0, 0, causal, scale, out, lse, nullptr, workspace,
                    workspace_bytes, nullptr, stream);
}

int bs_attn_varlen_fwd_noalloc(const bs_dims* dims, const void* q, const void* k, const void* v,
                               const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k,
                               int32_t num_seqs, int32_t max_seqlen, int causal, float scale,
                               void* out, float* lse, void* stream) {
  BS_TRY(check_dims(dims, true));
  BS_TRY(check_varlen_args(BS_OP_VARLEN_FWD, cu_seqlens_q, cu_seqlens_k, nullptr, nullptr,
                           num_seqs, max_seqlen));
  const size_t need = layout_of(BS_OP_VARLEN_FWD, *dims, num_seqs, max_seqlen).extra;
  if (need > kNoAllocScratchBytes)
    return fail(BS_ERR_WORKSPACE,
                "these sizes need %zu bytes of plan scratch, more than the %zu bytes of the "
                "allocation-free forward (use bs_attn_varlen_fwd with a workspace)",
                need, kNoAllocScratchBytes);
  void* ws = nullptr;
  BS_TRY(noalloc_scratch(stream, &ws));
  return fwd_common(BS_OP_VARLEN_FWD, dims, q, k, v, cu_seqlens_q, cu_seqlens_k, nullptr, nullptr,
                    num_seqs, max_seqlen, 0, 0, causal, scale, out, lse, nullptr, ws,
                    kNoAllocScratchBytes, static_cast<char*>(ws) + kNoAllocScratchBytes, stream);
}

int bs_attn_varlen_bwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                       const void* out, const float* lse, const void* dout,
                       const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k, int32_t num_seqs,
                       int32_t max_seqlen, int causal, float scale, void* dq, void* dk, void* dv,
                       void* workspace, size_t workspace_bytes, void* stream) {
  return bwd_common(BS_OP_VARLEN_BWD, dims, q, k, v, out, lse, dout, cu_seqlens_q, cu_seqlens_k,
                    nullptr, nullptr, num_seqs, max_seqlen, 0, 0, causal, scale, nullptr, dq, dk,
                    dv, 0, workspace, workspace_bytes, stream);
}

int bs_attn_chunk_fwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                      int64_t q_pos_offset, int64_t k_pos_offset, int causal, float scale,
                      void* out, float* lse, void* workspace, size_t workspace_bytes,
                      void* stream) {
  return fwd_common(BS_OP_CHUNK_FWD, dims, q, k, v, nullptr, nullptr, nullptr, nullptr, 1, 0,
                    q_pos_offset, k_pos_offset, causal, scale, out, lse, nullptr, workspace,
                    workspace_bytes, nullptr, stream);
}

int bs_attn_chunk_fwd_merge(const bs_dims* dims, const void* q, const void* k, const void* v,
                            int64_t q_pos_offset, int64_t k_pos_offset, int causal, float scale,
                            float* o_run, float* lse_run, int accumulate, void* out,
                            void* workspace, size_t workspace_bytes, void* stream) {
  const FwdMerge m{o_run, lse_run, accumulate != 0};
  return fwd_common(BS_OP_CHUNK_FWD, dims, q, k, v, nullptr, nullptr, nullptr, nullptr, 1, 0,
                    q_pos_offset, k_pos_offset, causal, scale, out, nullptr, &m, workspace,
                    workspace_bytes, nullptr, stream);
}

int bs_attn_chunk_bwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                      const void* out_merged, const float* lse_merged, const void* dout,
                      int64_t q_pos_offset, int64_t k_pos_offset, int causal, float scale,
                      float* dq_accum, void* dk, void* dv, int kv_accumulate, void* workspace,
                      size_t workspace_bytes, void* stream) {
  return bwd_common(BS_OP_CHUNK_BWD, dims, q, k, v, out_merged, lse_merged, dout, nullptr, nullptr,
                    nullptr, nullptr, 1, 0, q_pos_offset, k_pos_offset, causal, scale, dq_accum,
                    nullptr, dk, dv, kv_accumulate != 0, workspace, workspace_bytes, stream);
}

int bs_attn_packed_chunk_fwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                             const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k,
                             const int64_t* q_pos, const int64_t* k_pos, int32_t num_seqs,
                             int32_t max_seqlen, int causal, float scale, void* out, float* lse,
                             void* workspace, size_t workspace_bytes, void* stream) {
  return fwd_common(BS_OP_PACKED_CHUNK_FWD, dims, q, k, v, cu_seqlens_q, cu_seqlens_k, q_pos,
                    k_pos, num_seqs, max_seqlen, 0, 0, causal, scale, out, lse, nullptr,
                    workspace, workspace_bytes, nullptr, stream);
}

int bs_attn_packed_chunk_fwd_merge(const bs_dims* dims, const void* q, const void* k,
                                   const void* v, const int32_t* cu_seqlens_q,
                                   const int32_t* cu_seqlens_k, const int64_t* q_pos,
                                   const int64_t* k_pos, int32_t num_seqs, int32_t max_seqlen,
                                   int causal, float scale, float* o_run, float* lse_run,
                                   int accumulate, void* out, void* workspace,
                                   size_t workspace_bytes, void* stream) {
  const FwdMerge m{o_run, lse_run, accumulate != 0};
  return fwd_common(BS_OP_PACKED_CHUNK_FWD, dims, q, k, v, cu_seqlens_q, cu_seqlens_k, q_pos,
                    k_pos, num_seqs, max_seqlen, 0, 0, causal, scale, out, nullptr, &m,
                    workspace, workspace_bytes, nullptr, stream);
}

int bs_attn_packed_chunk_bwd(const bs_dims* dims, const void* q, const void* k, const void* v,
                             const void* out_merged, const float* lse_merged, const void* dout,
                             const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k,
                             const int64_t* q_pos, const int64_t* k_pos, int32_t num_seqs,
                             int32_t max_seqlen, int causal, float scale, float* dq_accum,
                             void* dk, void* dv, int kv_accumulate, void* workspace,
                             size_t workspace_bytes, void* stream) {
  return bwd_common(BS_OP_PACKED_CHUNK_BWD, dims, q, k, v, out_merged, lse_merged, dout,
                    cu_seqlens_q, cu_seqlens_k, q_pos, k_pos, num_seqs, max_seqlen, 0, 0, causal,
                    scale, dq_accum, nullptr, dk, dv, kv_accumulate != 0, workspace,
                    workspace_bytes, stream);
}

int bs_dq_finalize(const bs_dims* dims, const float* dq_accum, void* dq, void* stream) {
  BS_TRY(check_dims(dims, false));
  const int64_t qn = dims->total_q * dims->hq * dims->head_dim;
  BS_TRY(check_ptr(dq_accum, qn, "dq_accum"));
  BS_TRY(check_ptr(dq, qn, "dq"));
  ProfScope ps(BS_KERNEL_FINALIZE, static_cast<hipStream_t>(stream));
  BS_HIP(launch_dq_finalize(*dims, dq_accum, dq, static_cast<hipStream_t>(stream)),
         "dQ finalize launch");
  return ok();
}

int bs_lse_merge(const bs_dims* dims, const void* out_partials, const float* lse_partials,
                 int32_t n, void* out, float* lse, void* stream) {
  BS_TRY(check_dims(dims, false));
  if (n < 1) return fail(BS_ERR_INVALID_ARG, "n = %d must be >= 1", n);
  const int64_t qn = dims->total_q * dims->hq * dims->head_dim;
  BS_TRY(check_ptr(out_partials, qn * n, "out_partials"));
  BS_TRY(check_ptr(lse_partials, dims->total_q * dims->hq * n, "lse_partials"));
  BS_TRY(check_ptr(out, qn, "out"));
  BS_TRY(check_ptr(lse, dims->total_q * dims->hq, "lse"));
  ProfScope ps(BS_KERNEL_MERGE, static_cast<hipStream_t>(stream));
  BS_HIP(launch_lse_merge(*dims, out_partials, lse_partials, n, out, lse,
                          static_cast<hipStream_t>(stream)),
         "merge launch");
  return ok();
}

int bs_copy_async(void* dst, const void* src, size_t bytes, void* stream) {
  if (bytes == 0) return ok();
  if (dst == nullptr || src == nullptr) return fail(BS_ERR_INVALID_ARG, "dst or src is NULL");
  if (bytes > (size_t)INT64_MAX || overlaps(dst, (int64_t)bytes, src, (int64_t)bytes))
    return fail(BS_ERR_INVALID_ARG, "dst and src overlap");
  BS_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDeviceNoCU,
                        static_cast<hipStream_t>(stream)),
         "DMA copy");
  return ok();
}

int bs_softmax_xent(int64_t rows, int64_t vocab, int dtype, const void* logits,
                    const int64_t* labels, int64_t ignore_index, float grad_scale, float* loss,
                    float* lse, void* dlogits, void* stream) {
  if (dtype != BS_F32 && dtype != BS_BF16)
    return fail(BS_ERR_UNSUPPORTED, "dtype %d is not BS_F32 or BS_BF16", dtype);
  if (rows < 0 || rows >= kMaxTokens)
    return fail(BS_ERR_INVALID_ARG, "rows = %lld out of [0, 2^30)", (long long)rows);
  if (vocab < 1 || vocab > INT32_MAX)
    return fail(BS_ERR_INVALID_ARG, "vocab = %lld out of [1, 2^31)", (long long)vocab);
  if (!isfinite(grad_scale)) return fail(BS_ERR_INVALID_ARG, "grad_scale must be finite");
  if (rows == 0) return ok();
  if (logits == nullptr || labels == nullptr || loss == nullptr)
    return fail(BS_ERR_INVALID_ARG, "logits, labels or loss is NULL");
  const int64_t esize = dtype == BS_BF16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(logits) % esize != 0 ||
      (dlogits != nullptr && reinterpret_cast<uintptr_t>(dlogits) % esize != 0))
    return fail(BS_ERR_INVALID_ARG, "logits / dlogits not aligned to their element size");
  if (reinterpret_cast<uintptr_t>(labels) % 8 != 0 || reinterpret_cast<uintptr_t>(loss) % 4 != 0 ||
      (lse != nullptr && reinterpret_cast<uintptr_t>(lse) % 4 != 0))
    return fail(BS_ERR_INVALID_ARG, "labels / loss / lse not aligned to their element size");
  if (rows > INT64_MAX / esize / vocab)
    return fail(BS_ERR_INVALID_ARG, "rows * vocab elements exceed the address range");
  const int64_t nbytes = rows * vocab * esize;
  if (dlogits != nullptr && dlogits != logits && overlaps(dlogits, nbytes, logits, nbytes))
    return fail(BS_ERR_INVALID_ARG, "dlogits overlaps logits without being equal to it");
  ProfScope ps(BS_KERNEL_XENT, static_cast<hipStream_t>(stream));
  BS_HIP(launch_softmax_xent(rows, vocab, dtype, logits, labels, ignore_index, grad_scale, loss,
                             lse, dlogits, static_cast<hipStream_t>(stream)),
         "cross-entropy launch");
  return ok();
}

int bs_read_device_status(const void* workspace, void* stream) {
  if (workspace == nullptr) return fail(BS_ERR_WORKSPACE, "workspace is NULL");
  WsHeader h;
  hipStream_t s = static_cast<hipStream_t>(stream);
  BS_HIP(hipMemcpyAsync(&h, workspace, sizeof(h), hipMemcpyDeviceToHost, s), "status copy");
  BS_HIP(hipStreamSynchronize(s), "status sync");
  if (h.status != BS_DEV_OK)
    return fail(BS_ERR_DEVICE_STATUS, "device planner rejected cu_seqlens: code %d", h.status);
  return ok();
}

int bs_attn_plan_export(int op, const bs_dims* dims, const int32_t* cu_seqlens_q,
                        const int32_t* cu_seqlens_k, int32_t num_seqs, int32_t max_seqlen,
                        int64_t q_pos_offset, int64_t k_pos_offset, const int64_t* q_pos,
                        const int64_t* k_pos, int causal, void* workspace,
                        size_t workspace_bytes, int32_t* host_items, size_t capacity,
                        size_t* count, int32_t* tile_m, int32_t* tile_n, void* stream) {
  if (!valid_op(op)) return fail(BS_ERR_UNSUPPORTED, "unknown op %d", op);
  BS_TRY(check_dims(dims, true));
  if (count == nullptr || (capacity > 0 && host_items == nullptr))
    return fail(BS_ERR_INVALID_ARG, "count / host_items is NULL");
  const bool varlen = is_varlen(op);
  if (varlen)
    BS_TRY(check_varlen_args(op, cu_seqlens_q, cu_seqlens_k, q_pos, k_pos, num_seqs, max_seqlen));
  const WsLayout L = layout_of(op, *dims, varlen ? num_seqs : 1, max_seqlen);
  BS_TRY(check_ws(L, workspace, workspace_bytes));
  hipStream_t s = static_cast<hipStream_t>(stream);
  // the plan the op's main kernel walks: the last one of the op
  PlanCfg cfg[2];
  const int np = plans_of(op, *dims, cfg);
  WsLayout Lp;
  BS_HIP(run_plan(op, *dims, np - 1, cu_seqlens_q, cu_seqlens_k, q_pos, k_pos, num_seqs,
                  max_seqlen, q_pos_offset, k_pos_offset, causal, workspace, L, &Lp, s),
         "planner launch");
  WsHeader h;
  BS_HIP(hipMemcpyAsync(&h, workspace, sizeof(h), hipMemcpyDeviceToHost, s), "plan copy");
  BS_HIP(hipStreamSynchronize(s), "plan sync");
  if (h.status != BS_DEV_OK)
    return fail(BS_ERR_DEVICE_STATUS, "device planner rejected cu_seqlens: code %d", h.status);
  const size_t n = (size_t)h.n_items;
  *count = n;
  if (tile_m) *tile_m = cfg[np - 1].kind == kPlanFwd ? cfg[np - 1].tile_a : cfg[np - 1].tile_b;
  if (tile_n) *tile_n = cfg[np - 1].kind == kPlanFwd ? cfg[np - 1].tile_b : cfg[np - 1].tile_a;
  const size_t m = n < capacity ? n : capacity;
  if (m > 0) {
    std::vector<WorkItem> items(m);
    BS_HIP(hipMemcpyAsync(items.data(), static_cast<char*>(workspace) + L.sorted,
                          m * sizeof(WorkItem), hipMemcpyDeviceToHost, s),
           "plan copy");
    BS_HIP(hipStreamSynchronize(s), "plan sync");
    for (size_t i = 0; i < m; ++i) {
      const WorkItem& w = items[i];
      int32_t* o = host_items + 12 * i;
      const int32_t common[6] = {w.seg, w.tile, w.a_start, w.a_rows, w.b_start, w.b_len};
      memcpy(o, common, sizeof(common));
      if (cfg[np - 1].kind == kPlanFwd) {
        o[6] = w.n0; o[7] = w.n1; o[8] = w.diag; o[9] = 0;
      } else {
        o[6] = w.n0; o[7] = w.n1; o[8] = w.n2; o[9] = w.diag;
      }
      o[10] = 0;
      o[11] = 0;
    }
  }
  return ok();
}

int bs_set_profiling(int enable) {
  Profiler& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  for (auto& v : P.recs) {
    for (auto& pr : v) {
      hipEventSynchronize(pr.second);
      P.spare.push_back(pr.first);
      P.spare.push_back(pr.second);
    }
    v.clear();
  }
  P.on.store(enable != 0);
  return ok();
}

int bs_profile_read(int kind, double* total_ms, int64_t* launches) {
  if (kind < 0 || kind >= BS_KERNEL_COUNT) return fail(BS_ERR_INVALID_ARG, "unknown kernel kind %d", kind);
  if (total_ms == nullptr || launches == nullptr) return fail(BS_ERR_INVALID_ARG, "NULL output");
  Profiler& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  double sum = 0.0;
  for (auto& pr : P.recs[kind]) {
    BS_HIP(hipEventSynchronize(pr.second), "event sync");
    float ms = 0.f;
    BS_HIP(hipEventElapsedTime(&ms, pr.first, pr.second), "event elapsed");
    sum += ms;
  }
  *total_ms = sum;
  *launches = (int64_t)P.recs[kind].size();
  return ok();
}

const char* bs_last_error(void) { return g_err; }

}  // extern "C"
