// Definitions of the attention path of libbs_attn.so (gfx950 only): the ordered work
// list and its workspace, tile shapes, the placement of blocks on the XCDs, the
// swizzled LDS tiles with their copy and transposing reads, and the host launchers.
#pragma once

#include "common.hpp"

namespace bs {

constexpr int kDiagClamp = 1 << 30;

// One entry of the ordered work list (12 int32 = 48 bytes).
// Forward (query tile):  seg, tile=qtile, a_start=q_start, a_rows=q_rows,
//                        b_start=k_start, b_len=k_len, n0=n_full, n1=n_tiles, diag.
// Backward (key tile):   seg, tile=ktile, a_start=k_start, a_rows=k_rows,
//                        b_start=q_start, b_len=q_len, n0=qt_first, n1=n_masked,
//                        n2=n_vis, diag.
// Both: run0 = list slot of the first item of the segment, nrun = the segment's item
// count (the items of a segment are contiguous in the list).
struct WorkItem {
  int32_t seg, tile, a_start, a_rows, b_start, b_len, n0, n1, n2, diag, run0, nrun;
};
static_assert(sizeof(WorkItem) == 48, "work item is 12 int32");

enum PlanKind { kPlanFwd = 0, kPlanBwd = 1 };

// Tile sizes of each kernel family.  The forward walks query tiles of kFwdBM rows
// over key tiles of kFwdBN keys; the backward walks key tiles of kBwdBN keys over
// query tiles of bwd_bm(head_dim) rows: 96 at head_dim 128, 64 at head_dim 64 (a
// 96-row tile of 64-wide rows is 12 copy instructions, which 8 waves cannot share
// evenly).  The float32 kernels use their own sizes: 64 queries over 128-key tiles, and 32
// keys over 128-query tiles.
constexpr int kFwdBM = 128, kFwdBN = 64;
constexpr int kBwdBN = 128;
__host__ __device__ constexpr int bwd_bm(int head_dim) { return head_dim == 128 ? 96 : 64; }
constexpr int kF32BM = 64, kF32BN = 128;
constexpr int kF32BwdBN = 32, kF32BwdBM = 128;

// Workspace header: status word and item count, then the per-segment item
// offsets (segment order) and first slots (list order), the ordered work list,
// then op-specific float buffers.
struct WsHeader {
  int32_t status;
  int32_t n_items;
  int32_t pad[62];
};

// The dK/dV kernel walks a segment one head at a time from this many streamed rows (b_len)
// on; the forward and dQ kernels do so for every segment.
constexpr int kHeadMajorRowsDkdv = 16384;

// Work item and head of block b of a grid of n_items * n_heads blocks; false when it has none.
// Blocks are dealt to the 8 XCDs round-robin (block b runs on XCD b % 8), so with n_heads a
// multiple of 8 each XCD owns the hx = n_heads / 8 heads x*hx .. x*hx+hx-1 and walks the list
// segment by segment.  Inside a segment's run its heads are interleaved item by item, except where
// the segment streams at least min_rows rows and the XCD's heads read more than one stream (hx >
// heads_per_stream: heads that share a KV head share its K/V stream): there the XCD walks one
// head's items at a time, so that the workgroups resident on it read one stream, not hx /
// heads_per_stream, and each tile of it comes into the XCD's L2 that many times less often.
//
// The item is read beside the list's length, except with kCountFirst, where it is read after it: on
// long chunks that small difference in when workgroups start decides how far apart those that share
// a K/V stream drift (a 32K-token query chunk against 32K-key chunks, 32/32 heads, HBM reads per
// launch over several GPUs, beside / after: dQ 8.5 to 9.3 / 6.4 GB, forward 6.4 to 7.6 / 7.4 to 10.7,
// dK/dV 4.7 / 4.7; dQ 20.92 / 20.61 ms).
template <bool kCountFirst = false>
__device__ __forceinline__ bool block_work(int b, const WsHeader* __restrict__ hdr,
                                           const WorkItem* __restrict__ items, int n_heads,
                                           int heads_per_stream, int min_rows, WorkItem& it,
                                           int& head) {
  const int n_items = hdr->n_items;
  if ((n_heads & 7) != 0) {
    const int i = b / n_heads;
    if (i >= n_items) return false;
    it = items[i];
    head = b - i * n_heads;
    return true;
  }
  const int hx = n_heads >> 3, jb = b >> 3;
  const int g = jb / hx;
  WorkItem gi;
  if constexpr (!kCountFirst) gi = items[g];  // (g is inside the list's room)
  if (g >= n_items) return false;
  if constexpr (kCountFirst) gi = items[g];
  const int r = jb - gi.run0 * hx;  // 0 <= r < nrun * hx: this block's place in the run
  int i, hl;
  if (hx > heads_per_stream && gi.b_len >= min_rows) {
    hl = r / gi.nrun;
    i = gi.run0 + (r - hl * gi.nrun);
  } else {
    i = g;
    hl = r - (g - gi.run0) * hx;
  }
  it = i == g ? gi : items[i];
  head = (b & 7) * hx + hl;
  return true;
}

// Segment b of the problem: query start/length, key start/length, diagonal.
struct Seg {
  int64_t q0, lq, k0, lk;
  int32_t diag;
};

__device__ __forceinline__ int32_t clamp_diag(int64_t d) {
  return (int32_t)(d < -kDiagClamp ? -kDiagClamp : (d > kDiagClamp ? kDiagClamp : d));
}

// Diagonal: key j visible to query i iff j - i <= diag.  Varlen segments are
// aligned bottom-right (diag = len_k - len_q); packed chunk segments and single
// chunks take it from the global positions of their first query and key.
__device__ __forceinline__ Seg load_seg(const int32_t* cu_q, const int32_t* cu_k,
                                        const int64_t* q_pos, const int64_t* k_pos, int32_t b,
                                        int64_t total_q, int64_t total_k, int32_t diag_chunk) {
  Seg s;
  if (cu_q == nullptr) {  // chunk mode: one segment, diagonal from the offsets
    s.q0 = 0; s.lq = total_q; s.k0 = 0; s.lk = total_k; s.diag = diag_chunk;
  } else {
    s.q0 = cu_q[b]; s.lq = (int64_t)cu_q[b + 1] - cu_q[b];
    s.k0 = cu_k[b]; s.lk = (int64_t)cu_k[b + 1] - cu_k[b];
    s.diag = q_pos == nullptr ? clamp_diag(s.lk - s.lq) : clamp_diag(q_pos[b] - k_pos[b]);
  }
  return s;
}

// Work item `tile` of segment b (run0, nrun: its segment's run in the list).
__device__ __forceinline__ WorkItem make_item(const Seg& s, int32_t b, int64_t tile, int causal,
                                              int kind, int tile_a, int tile_b, int32_t run0,
                                              int32_t nrun) {
  const int64_t diag = s.diag;
  WorkItem w;
  w.seg = b; w.tile = (int32_t)tile; w.diag = s.diag; w.run0 = run0; w.nrun = nrun;
  if (kind == kPlanFwd) {
    const int64_t BM = tile_a, BN = tile_b;
    const int64_t q_first = tile * BM;
    const int64_t q_last = (q_first + BM < s.lq ? q_first + BM : s.lq) - 1;
    const int64_t nkt = (s.lk + BN - 1) / BN;
    int64_t n_tiles, n_full;
    if (causal) {
      const int64_t lim = q_last + diag;
      n_tiles = lim < 0 ? 0 : (lim / BN + 1 < nkt ? lim / BN + 1 : nkt);
      int64_t f = q_first + diag + 1;
      f = f < s.lk ? f : s.lk;
      n_full = f > 0 ? f / BN : 0;
    } else {
      n_tiles = nkt;
      n_full = s.lk / BN;
    }
    w.a_start = (int32_t)(s.q0 + q_first);
    w.a_rows = (int32_t)(q_last - q_first + 1);
    w.b_start = (int32_t)s.k0;
    w.b_len = (int32_t)s.lk;
    w.n0 = (int32_t)n_full;
    w.n1 = (int32_t)n_tiles;
    w.n2 = (int32_t)n_tiles;
  } else {
    const int64_t BM = tile_b, BN = tile_a;
    const int64_t k_first = tile * BN;
    const int64_t nqt = (s.lq + BM - 1) / BM;
    const bool in_range = k_first + BN <= s.lk;
    int64_t first, ffirst;
    if (causal) {
      const int64_t r = k_first - diag;  // first query row that sees key k_first
      first = r > s.lq - 1 ? nqt : (r > 0 ? r / BM : 0);
      if (!in_range) {
        ffirst = nqt;
      } else {
        const int64_t t = k_first + BN - 1 - diag;  // FULL needs q_first >= t
        ffirst = t <= 0 ? 0 : (t + BM - 1) / BM;
        ffirst = ffirst < nqt ? ffirst : nqt;
      }
    } else {
      first = 0;
      ffirst = in_range ? 0 : nqt;
    }
    const int64_t n_vis = nqt - first;
    const int64_t n_masked = ffirst - first > 0 ? ffirst - first : 0;
    w.a_start = (int32_t)(s.k0 + k_first);
    w.a_rows = (int32_t)(s.lk - k_first < BN ? s.lk - k_first : BN);
    w.b_start = (int32_t)s.q0;
    w.b_len = (int32_t)s.lq;
    w.n0 = (int32_t)first;
    w.n1 = (int32_t)n_masked;
    w.n2 = (int32_t)n_vis;
  }
  return w;
}

// What a kernel needs to find its own work item (no planning launch), for grids that the chip
// holds at once (about: the rule is in capi.hip): a workgroup reads cu_seqlens about as fast as a
// work item.
constexpr int kSelfMaxSegs = 256;
// Up to so many segments are walked in the planner's order; more of them, as they are stored: each is
// then short, and ranking them costs more than the order gives (forward, us, ranked / as stored: 238
// segments of one query over 179 keys on average, 1/1 heads, 15.0 / 10.8; 107 segments, 25.7K tokens, 2/2
// heads, head_dim 64: 15.0 / 15.4).
constexpr int kSelfRankSegs = 64;
struct PlanArgs {
  const int32_t* cu_q;  // NULL: one chunk with diagonal diag_chunk
  const int32_t* cu_k;
  const int64_t* q_pos;
  const int64_t* k_pos;
  WsHeader* hdr;
  int64_t total_q, total_k;
  int32_t num_seqs, max_seqlen, diag_chunk;
};
// LDS of self_plan.
struct SelfLds {
  __attribute__((aligned(16))) uint2 seg[kSelfRankSegs];  // size (len_q + len_k) and items of each segment
  uint32_t at[kSelfRankSegs];  // slots before it (more segments: items of each wave's)
  int32_t bad, n;
  int32_t found, slot, items;  // the segment of item i, its first slot and its items
};

// Head and list slot (x splits) of block b.  With `own` (and n_heads a multiple of 8) each XCD owns
// a contiguous eighth of the heads, as block_work deals them, so that the query heads of a KV group
// read its K and V into one L2; otherwise the heads go round.  `own` where no chain is split, as in
// the list (forward, 512 queries over 16K keys, 32/32 heads, head_dim 128: round 239 us, own 230),
// and of the split ones where heads share 256-byte rows (6 segments of 12..28 queries over 3..9K
// keys, 48/8 heads, head_dim 128: round 148, own 114).  Split chains of head_dim 64, or without a
// group, do not gain (256 queries over 8K keys, 32/4 heads, head_dim 64: round 40.7, own 43.2; 3
// queries over 6.4K keys, 32/32: 26.7, 28.7).
__device__ __forceinline__ int self_block(int b, int n_heads, bool own, int& head) {
  if (!own || (n_heads & 7) != 0) {
    const int i = b / n_heads;
    head = b - i * n_heads;
    return i;
  }
  const int hx = n_heads >> 3, jb = b >> 3, i = jb / hx;
  head = (b & 7) * hx + (jb - i * hx);
  return i;
}

// Item i of the list, in the planner's order (larger segments first up to kSelfRankSegs of them, a
// segment's longest chains first), for a workgroup of at least kSelfMaxSegs threads; false when
// there is none or cu_seqlens is rejected.  The order matters on grids that the chip holds at once
// too: it decides which workgroups share a CU (forward, us, planning launch and list / segments and
// tiles as they come / in order: 300 queries each over 2.3K and 6.3K keys, 48/8 heads, head_dim 64, 74 / 84 / 70; 4,096
// tokens, 12/4, head_dim 64, 54 / 57 / 49).  Block 0 writes the header.
__device__ __forceinline__ bool self_plan(const PlanArgs& a, int causal, int kind, int tile_a,
                                          int tile_b, int32_t i, SelfLds& lds, WorkItem& it) {
  const int tid = threadIdx.x;
  if (a.cu_q == nullptr) {
    const Seg s = load_seg(nullptr, nullptr, nullptr, nullptr, 0, a.total_q, a.total_k, a.diag_chunk);
    const int32_t n = (int32_t)(((kind == kPlanFwd ? s.lq : s.lk) + tile_a - 1) / tile_a);
    if (blockIdx.x == 0 && tid == 0) {
      a.hdr->status = BS_DEV_OK;
      a.hdr->n_items = n;
    }
    if (i >= n) return false;
    it = make_item(s, 0, kind == kPlanFwd ? n - 1 - i : i, causal, kind, tile_a, tile_b, 0, n);
    return true;
  }
  if (tid == 0) {
    lds.bad = BS_DEV_OK;
    lds.n = 0;
  }
  if (tid < kSelfRankSegs) lds.at[tid] = 0;
  __syncthreads();
  uint2 mine = {0, 0};
  if (tid < a.num_seqs) {
    const Seg s = load_seg(a.cu_q, a.cu_k, nullptr, nullptr, tid, a.total_q, a.total_k, 0);
    if (s.lq < 0 || s.lk < 0) atomicCAS(&lds.bad, 0, BS_DEV_NOT_MONOTONE);
    else if (s.lq > a.max_seqlen || s.lk > a.max_seqlen) atomicCAS(&lds.bad, 0, BS_DEV_TOO_LONG);
    else mine = {(uint32_t)(s.lq + s.lk), (uint32_t)(((kind == kPlanFwd ? s.lq : s.lk) + tile_a - 1) / tile_a)};
  }
  if (tid < kSelfRankSegs) lds.seg[tid] = mine;
  if (tid == 0) {
    if (a.cu_q[0] != 0 || a.cu_k[0] != 0) atomicExch(&lds.bad, BS_DEV_BAD_FIRST);
    else if (a.cu_q[a.num_seqs] != a.total_q || a.cu_k[a.num_seqs] != a.total_k)
      atomicExch(&lds.bad, BS_DEV_BAD_TOTAL);
  }
  __syncthreads();
  if (a.num_seqs <= kSelfRankSegs) {
    // slots before segment b: the entries [j, end) of the table eight at a time, so that their
    // (broadcast) reads are under way together; entries past num_seqs are empty
    const int b = tid & 63;
    uint32_t at = 0, n = 0;
    auto rank = [&](int j, int end) {
      const uint32_t size = lds.seg[b].x;
      for (; j < end; j += 8) {
        uint4 o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = reinterpret_cast<const uint4*>(lds.seg)[(j >> 1) + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // equal sizes in their own order
          n += o[u].y + o[u].w;
          at += o[u].x + (j + 2 * u < b ? 1u : 0u) > size ? o[u].y : 0u;
          at += o[u].z + (j + 2 * u + 1 < b ? 1u : 0u) > size ? o[u].w : 0u;
        }
      }
    };
    if (a.num_seqs <= 16) {  // one wave: sharing the table costs more (0.4 us at two segments)
      if (tid < 64) rank(0, a.num_seqs);
      if (tid == 0) lds.n = (int32_t)n;
    } else {  // each wave a part of it
      const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
      const int len = ((a.num_seqs - 1) / (int)(blockDim.x >> 6) + 8) & ~7;
      rank(w * len, min(a.num_seqs, (w + 1) * len));
      atomicAdd(&lds.at[b], at);
      if (b == 0) atomicAdd(&lds.n, (int32_t)n);
      __syncthreads();
      at = lds.at[b];
    }
    if (tid < a.num_seqs && (uint32_t)i - at < mine.y) {  // (at most one segment)
      lds.found = tid;
      lds.items = (int32_t)mine.y;
      lds.slot = (int32_t)at;
    }
  } else {  // as they are stored
    uint32_t run = mine.y;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t x = __shfl_up(run, off);
      run += (tid & 63) >= off ? x : 0;
    }
    if ((tid & 63) == 63) lds.at[tid >> 6] = run;
    __syncthreads();
    uint32_t at = run - mine.y, n = 0;
    for (int w = 0; w < kSelfMaxSegs / 64; ++w) {
      at += w < (tid >> 6) ? lds.at[w] : 0;
      n += lds.at[w];
    }
    if (tid == 0) lds.n = (int32_t)n;
    if (tid < a.num_seqs && (uint32_t)i - at < mine.y) {
      lds.found = tid;
      lds.items = (int32_t)mine.y;
      lds.slot = (int32_t)at;
    }
  }
  __syncthreads();
  const int32_t code = lds.bad, n = lds.n;
  if (blockIdx.x == 0 && tid == 0) {
    a.hdr->status = code;
    a.hdr->n_items = code == BS_DEV_OK ? n : 0;
  }
  if (code != BS_DEV_OK || i >= n) return false;  // uniform
  const int32_t b = lds.found, at = lds.slot, cnt = lds.items;
  const Seg s = load_seg(a.cu_q, a.cu_k, a.q_pos, a.k_pos, b, a.total_q, a.total_k, 0);
  it = make_item(s, b, kind == kPlanFwd ? cnt - 1 - (i - at) : i - at, causal, kind, tile_a, tile_b, at, cnt);
  return true;
}

struct WsLayout {
  size_t seg_off;     // int32[num_seqs + 1]
  size_t seg_dst;     // int32[num_seqs]
  size_t sorted;      // WorkItem[max_items]
  size_t dvec;        // float[hq * T]      (backward: rowsum(dO * O))
  size_t dq_late;     // float[T * hq * d]  (float32 varlen backward: dq that lies over an input)
  size_t extra;       // pieces of the few-query forward, or partials of split chains: optional
  size_t total;
  int64_t max_items;
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Operand of a 32x32x16 bf16 MFMA that is the TRANSPOSE of a row-major LDS tile.
//
// X is a row-major bf16 tile in LDS (`stride` elements per row) whose rows run
// along the MFMA contraction index and whose columns run along the MFMA row
// (A operand) / column (B operand) index.  Lane l = 32*hh + c receives
// X[k0 + (e/4)*8 + hh*4 + e%4][m0 + c] as element e (e = 0..7): inside every
// 16-step of the contraction, lanes 0-31 take rows 0-3 and 8-11, lanes 32-63
// rows 4-7 and 12-15.  That is exactly the contraction order in which a lane
// holds the rows of a 32x32 MFMA result, so a result kept in registers (P, dS)
// can be fed as the other operand without reshuffling.
//
// Built from two ds_read_b64_tr_b16: inside each 16-lane group, output lane i
// gets element (i % 4) of the 8-byte chunk addressed by lane 4e + i/4, for
// e = 0..3; so lane s addresses row k0 + r*8 + hh*4 + (s%16)/4, columns
// m0 + 16*((s/16)%2) + 4*(s%4) .. +3, in read r = 0, 1.
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

__device__ __forceinline__ const bf16* tr_lane_ptr(const bf16* tile, int stride, int k0, int m0,
                                                   int lane) {
  const int i = lane & 15;
  return tile + (k0 + (lane >> 5) * 4 + (i >> 2)) * stride + m0 + ((lane >> 4) & 1) * 16 + (i & 3) * 4;
}

// The operand from two lane addresses: rows k0 + hh*4 + (i/4) and the row 8 below.
__device__ __forceinline__ bf16x8 lds_read_tr2(const bf16* p0, const bf16* p1) {
  const i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p0));
  const i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p1));
  typedef short i16x8 __attribute__((ext_vector_type(8)));
  const i16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// `p` is tr_lane_ptr(tile, stride, k0, m0, lane) of a padded tile.
__device__ __forceinline__ bf16x8 lds_read_tr(const bf16* p, int stride) {
  return lds_read_tr2(p, p + 8 * stride);
}

// Swizzled row-major LDS tile with D bf16 per row (no padding) for tiles that are
// read both ways: row reads (16 consecutive rows, one 16-byte chunk each) and
// transposing reads (4 consecutive rows, 4 consecutive chunks each, per half
// wave).  Chunk c of row r is stored at chunk c ^ g(r).  With 64 banks of 4
// bytes, g makes both patterns conflict-free:
//   D = 128 (16 chunks = one bank line per row): g(r) = ((r&3) << 2) | ((r>>2)&3)
//     - any 16 consecutive rows: g is a bijection of r mod 16;
//     - 4 aligned rows: (r&3) moves each row's 4-chunk group to a different quarter.
//   D = 64 (8 chunks = half a bank line per row): g(r) = (((r>>1)&1) << 2) | ((r>>2)&3)
//     - rows of equal parity share a half line, and g is a bijection over them;
//     - of 4 aligned rows, the two of equal parity land in different 4-chunk groups.
// g depends on r mod 16 only, so tiles may be addressed from any 16-row boundary.
template <int D>
__device__ __forceinline__ int swz_g(int r) {
  static_assert(D == 64 || D == 128, "head_dim");
  return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
}

// Element offset of 16-byte chunk `c` of row `r`.
template <int D>
__device__ __forceinline__ int swz_off(int r, int c) {
  return r * D + ((c ^ swz_g<D>(r)) << 3);
}

// The swizzle only moves bits 4..7 of a byte offset inside a row (it XORs the chunk
// index), so a lane's reads of a tile differ by a lane-independent XOR plus a multiple of
// a row: one lane base per access pattern gives every address with one v_xor_b32, and the
// row part (and the tile's own LDS address) go into the instruction's immediate offset.
//   row read of chunk (2 kk + hh) of row (32 kb + c), lane = 32 hh + c:
//     swz_off(32 kb + c, 2 kk + hh) * 2 == (swz_row_base(lane) ^ (kk << 5)) + kb * 64 * D
//   transposing read r of contraction rows k0 = 16 ks, columns m0 = 32 db:
//     swz_tr_off(16 ks, 32 db, r, lane) * 2
//         == (swz_tr_base(lane) ^ ((db << 6) | (r << 5))) + ks * 32 * D + r * 16 * D
template <int D>
__device__ __forceinline__ int swz_row_base(int lane) {
  return swz_off<D>(lane & 31, lane >> 5) * 2;
}
template <int D>
__device__ __forceinline__ int swz_tr_base(int lane);

// One wave's share of copying rows 0..R-1 of a swizzled [R][D] bf16 tile from global
// memory straight into LDS (buffer_load_dwordx4 ... lds: lane l of an instruction
// writes 16 bytes at LDS base + offset + 16*l, so an instruction fills 64/(D/8) whole
// rows, 1 KB, and each lane fetches the global chunk that the swizzle places at its
// LDS position).  Row r of the tile comes from src + min(r, last) * gstride elements:
// rows past the end repeat the last valid one.  Completion is waited for with
// wait_vmem_all().
//
// Each wave copies a contiguous run of PER instructions from one LDS base (M0): the
// instruction offset (0, 1 KB, 2 KB, 3 KB) moves both the LDS and the global address,
// so the per-lane global offsets subtract it, and the buffer starts 4 KB before `src`
// to keep them non-negative (only src + row offsets are ever accessed).
//
// The buffer form (MUBUF) rather than global_load_lds (FLAT): the compiler treats a
// pending FLAT copy into LDS as a possible LDS access of unknown order and then
// waits for all LDS reads (lgkmcnt(0)) before every use, which defeats reading LDS
// operands ahead.  Byte offsets (R rows x gstride x 2 + 4 KB) stay below 2^31 for
// the head counts the C API accepts.
template <int K, int PER, int D, int AUX>
struct DmaRun {
  static __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, bf16* lds, int row0,
                                               int sub, int phys, int gstride, int last) {
    constexpr int RPI = 64 / (D / 8);
    const int row = row0 + K * RPI + sub;
    const int r = row < last ? row : last;
    const int voff = (r * gstride + ((phys ^ swz_g<D>(row)) << 3)) * 2 + 4096 - K * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16,
                                             voff, 0, K * 1024, AUX);
    DmaRun<K + 1, PER, D, AUX>::issue(rs, lds, row0, sub, phys, gstride, last);
  }
};
template <int PER, int D, int AUX>
struct DmaRun<PER, PER, D, AUX> {
  static __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t, bf16*, int, int, int, int,
                                               int) {}
};

// AUX: cache policy bits of the instruction (2: non-temporal).
template <int D, int R, int NWAVES, int AUX = 0>
__device__ __forceinline__ void dma_tile(bf16* lds_tile, const bf16* src, int gstride, int last,
                                         int wave, int lane) {
  constexpr int CPR = D / 8, RPI = 64 / CPR, NI = R / RPI, PER = NI / NWAVES;
  static_assert(NI % NWAVES == 0, "whole instructions per wave");
  static_assert(PER >= 1 && PER <= 4, "instruction offsets of one run fit in 12 bits");
  const int sub = lane / CPR, phys = lane % CPR;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(src) - 4096), 0, 0x7fffffff, 0x00020000);
  const int u0 = wave * PER;  // first instruction (1 KB of LDS) of this wave's run
  DmaRun<0, PER, D, AUX>::issue(rsrc, lds_tile + u0 * RPI * D, u0 * RPI, sub, phys, gstride, last);
}

// Element offset, in a swizzled tile, of this lane's 8-byte piece of the transposing
// read r (0 or 1) at contraction row k0 (a multiple of 16) and column m0 (a multiple
// of 32): row k0 + 8r + 4hh + i/4, column m0 + 16*((lane/16)%2) + 4*(i%4).
template <int D>
__device__ __forceinline__ int swz_tr_off(int k0, int m0, int r, int lane) {
  const int i = lane & 15;
  const int row = k0 + 8 * r + 4 * (lane >> 5) + (i >> 2);
  const int col = m0 + ((lane >> 4) & 1) * 16 + (i & 3) * 4;
  return swz_off<D>(row, col >> 3) + (col & 7);
}
template <int D>
__device__ __forceinline__ int swz_tr_base(int lane) {
  return swz_tr_off<D>(0, 0, 0, lane) * 2;
}
// Byte-addressed LDS views used with the bases above.
__device__ __forceinline__ bf16x8 lds_row16(const bf16* tile, int byte_off) {
  return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(tile) + byte_off);
}
__device__ __forceinline__ bf16x8 lds_tr16(const bf16* tile, int off0, int off1) {
  const char* t = reinterpret_cast<const char*>(tile);
  return lds_read_tr2(reinterpret_cast<const bf16*>(t + off0), reinterpret_cast<const bf16*>(t + off1));
}

}  // namespace bs

// Host-side launchers implemented in the .hip files (all enqueue on `stream`).
namespace bs {
// A second list planned by the same launch (up to kPlanFusedSegs segments): its header, the items
// right behind it.
constexpr int kPlanFusedSegs = 1024;
struct PlanSecond {
  PlanKind kind;
  int tile_a, tile_b;
  int64_t max_items;
  void* hdr;
};
static_assert(sizeof(WsHeader) == 256, "the items of a second list start aligned");
// Segments: cu_q/cu_k (NULL: one chunk with diagonal diag_chunk); q_pos/k_pos
// (NULL: diagonal len_k - len_q of each segment, else q_pos[b] - k_pos[b]).
hipError_t launch_plan(PlanKind kind, const int32_t* cu_q, const int32_t* cu_k,
                       const int64_t* q_pos, const int64_t* k_pos, int32_t num_seqs,
                       int64_t total_q, int64_t total_k, int32_t max_seqlen, int32_t diag_chunk,
                       int causal, int tile_a, int tile_b, int64_t max_items, void* ws,
                       const WsLayout& L, const PlanSecond* second, hipStream_t stream);

// Forward epilogue that folds the step into a running result instead of writing
// a partial (ring steps merged as they arrive): o_run float32 [T, hq, d], lse_run
// [hq, T] natural log; accumulate = 0 replaces the running state, otherwise the
// two are combined by their log-sum-exp weights.  With `out` non-null the merged
// output goes there in the input dtype and o_run is not written.
struct FwdMerge {
  float* o_run;
  float* lse_run;
  int accumulate;
};

// A grid that the chip holds at once: its workgroups plan for themselves (plan.hdr set), and
// `splits` of them share each work item's chain of tiles.  With splits > 1 every one leaves a
// float32 partial in `part` (slab s of splits; [rows][d] in the layout of the output, twice for
// dK and dV; the forward's followed by float2 (max in log2 units, sum) [splits][T * hq]) and a
// second kernel combines them.
struct SelfPlan {
  PlanArgs plan;
  int64_t items;  // work items at most
  int32_t splits;
  float* part;
};

// merge == NULL: plain forward writing (out, lse).  self == NULL: the work list in ws.
hipError_t launch_fwd_bf16(const bs_dims& dims, const void* q, const void* k, const void* v,
                           int causal, float scale, void* out, float* lse,
                           const FwdMerge* merge, const void* ws, const WsLayout& L,
                           const SelfPlan* self, hipStream_t stream);
// Combines the forward's partials into (out, lse) or the running state.
hipError_t launch_fwd_combine(const bs_dims& dims, const SelfPlan& self, void* out, float* lse,
                              const FwdMerge* merge, hipStream_t stream);
// out0 / out1 (one of them may be NULL) = sum of the slabs of n floats, slab s of out0 at part +
// s n, of out1 behind out0's: written as bf16 or float32, or added into float32.
enum SumOut { kSumBf16 = 0, kSumAddF32 = 1, kSumF32 = 2 };
hipError_t launch_sum_slabs(const float* part, int splits, int64_t n, void* out0, void* out1,
                            SumOut mode, const WsHeader* hdr, hipStream_t stream);
// The forward of segments of few queries (few_bf16.hip): no plan, buf of F.bytes, the header
// only for the status word.  cu_q, cu_k of at most kFewMaxSegs segments.
constexpr int kFewMaxSegs = 1024;
constexpr int kFewSlabs = 32;  // pieces of a row at most
struct FewLayout {
  size_t part, stat;  // offsets in buf of the pieces' sums and statistics (counts come first)
  size_t bytes;       // 0: the call does not take this path
  int32_t slabs;      // pieces of a row at most; 1: no row has two
  int32_t per_min;    // key blocks per workgroup at least, if a segment may have max_seqlen keys
  int32_t blocks;     // workgroups
};
constexpr int few_block_keys(int head_dim) { return head_dim == 128 ? 128 : 256; }
// Key blocks per workgroup with which rows of up to nkb blocks have at most `slabs` > 1 pieces (at
// most ceil(nkb / per) + 1 of them).
__host__ __device__ constexpr int32_t few_per_min(int32_t nkb, int32_t slabs) {
  return nkb > 1 ? (nkb + slabs - 2) / (slabs - 1) : 1;
}
hipError_t launch_few_fwd(const bs_dims& dims, const void* q, const void* k, const void* v,
                          const int32_t* cu_q, const int32_t* cu_k, int32_t num_seqs,
                          int32_t max_seqlen, int causal, float scale, void* out, float* lse,
                          void* hdr, void* buf, const FewLayout& F, hipStream_t stream);
// The bf16 dQ kernel also forms D = rowsum(dO * O) and stores it in dvec for the dK/dV
// kernel.
hipError_t launch_dq_bf16(const bs_dims& dims, const void* q, const void* k, const void* v,
                          const void* out, const void* dout, const float* lse, float* dvec,
                          int causal, float scale, void* dq, float* dq_acc, const void* ws,
                          const WsLayout& L, const SelfPlan* self, hipStream_t stream);
hipError_t launch_dkdv_bf16(const bs_dims& dims, const void* q, const void* k, const void* v,
                            const void* dout, const float* lse, const float* dvec, int causal,
                            float scale, void* dk, void* dv, int kv_accumulate, const void* ws,
                            const WsLayout& L, const SelfPlan* self, hipStream_t stream);

hipError_t launch_fwd_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                          int causal, float scale, void* out, float* lse, const FwdMerge* merge,
                          const void* ws, const WsLayout& L, hipStream_t stream);
// dq written (dq_accumulate == 0) or added into; like the bf16 kernel it stores D in dvec.
hipError_t launch_dq_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                         const void* out, const void* dout, const float* lse, float* dvec,
                         int causal, float scale, void* dq, int dq_accumulate, const void* ws,
                         const WsLayout& L, hipStream_t stream);
// splits > 1: each item's steps shared by that many workgroups, their sums in part (as SelfPlan).
hipError_t launch_dkdv_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                           const void* dout, const float* lse, const float* dvec, int causal,
                           float scale, void* dk, void* dv, int kv_accumulate, const void* ws,
                           const WsLayout& L, int splits,
                           float* part, hipStream_t stream);

hipError_t launch_dq_finalize(const bs_dims& dims, const float* dq_acc, void* dq,
                              hipStream_t stream);
hipError_t launch_lse_merge(const bs_dims& dims, const void* out_parts, const float* lse_parts,
                            int32_t n, void* out, float* lse, hipStream_t stream);
}  // namespace bs
