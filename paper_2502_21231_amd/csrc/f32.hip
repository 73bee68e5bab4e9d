// float32 attention kernels for gfx950 (forward, dQ, dK/dV): float32 operands and float32
// accumulation throughout, on the float32 matrix instruction v_mfma_f32_32x32x2_f32.
//
// That instruction occupies a SIMD's matrix core for 64 cycles per 4,096 FLOP (157 TFLOP/s
// over the chip; a plain library product reaches 151), sixteen times longer per FLOP than the
// bf16 one, so these kernels are bound by it and by how evenly the waves share it: the
// exponentials, the LDS reads (one 16-byte read feeds four products, 256 cycles) and the tile
// copies all hide under it.  The shapes are therefore chosen for the number of waves, not for
// data reuse:
//   forward, dQ  64 queries x 128-key tiles, 8 waves = 2 query blocks x 4 key blocks of 32;
//                each wave keeps its own running softmax (or dQ sum) over its key blocks, and
//                the four are combined through LDS once, at the end;
//   dK/dV        32 keys x 128-query tiles, 8 waves = 4 query blocks x 2 roles as in the bf16
//                kernel (S, P, dV / dP, dS, dK, with P handed over through LDS), the four query
//                blocks' sums combined at the end.
// A segment of n keys is then a chain of n/128 tiles instead of n/64 on one wave, and small
// batches still give every SIMD two waves.  A wave whose 32 x 32 block is masked throughout
// skips its products.
//
// Measured at 2,048 tokens in 5 segments, 8/4 heads, head_dim 64, against one thread per row
// on the vector unit before: forward 1,010 -> 35 us, dQ 880 -> 49 us, dK/dV 2,300 -> 84 us
// (10, 15 and 19 us of useful FLOP at the library product's rate: one segment holds half of the
// tokens, and the kernels wait for its chains of up to eight 128-row tiles); error of dK against
// float64 7.4e-7 -> 4.8e-7.  At 4,096 tokens, 32/8 heads, head_dim 128: 126 -> 2.5 ms for the three.  Few key tiles
// (a rule in capi.hip): several workgroups share a dK/dV item (751 tokens, 16/2 heads: 329 -> 165
// us forward + backward).
//
// Orientation, as in the bf16 kernels: the forward and dQ compute S^T = K Q^T (a lane owns one
// query and 16 of a block's 32 keys), dK/dV computes S = Q K^T (a lane owns one key).  The
// 32x32x2 operand of lane 32 hh + c is element [c][hh] of a 32 x 2 block, so
//   row operands (contraction over head_dim): a lane reads 16 bytes of its row, elements
//     8 kk + 4 hh .. + 3, which feed four products (the contraction order is permuted alike on
//     both sides);
//   column operands (contraction over the block's 32 rows): in the row order in which a lane
//     holds a result, row (r/4)*8 + hh*4 + r%4 in step r, so P and dS feed the product from
//     registers; a lane reads DB = D/32 consecutive floats of that row, columns DB c .., one
//     for each of the DB accumulators, whose column i is then head_dim index DB i + db.
// Both reads hit one tile in LDS: rows of D floats, 16-byte chunk k of row r stored at chunk
// k ^ (r & 15) (free of bank conflicts both ways), copied from HBM straight into LDS.  Rows
// past a segment are copied from its last valid row and masked.
#include "attn.hpp"

namespace bs {
namespace {

struct F32Params {
  const float* q;
  const float* k;
  const float* v;
  const float* dout;
  const float* out;  // dQ: the forward's output, for D = rowsum(dO * O)
  const float* lse;
  float* dvec;       // D: written by the dQ kernel, read by the dK/dV kernel
  float* o;
  float* lse_out;
  float* o_run;    // forward running-merge mode (non-null): running output
  float* lse_run;  // and its running LSE
  int32_t accumulate;
  float* dq;
  int32_t dq_accumulate;  // dQ added into (not written over) the output
  float* dk;
  float* dv;
  const WsHeader* hdr;
  const WorkItem* items;
  int64_t total_q;
  int32_t hq, hkv, group;
  int32_t causal;
  int32_t kv_accumulate;  // dK, dV added into (not written over) the outputs
  float scale, scale_log2;
  int32_t splits;  // dK/dV: workgroups of an item
  float* part;     // and, of several, where they leave their sums
  int64_t total_k;
};

typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Copy instructions K .. N-1 of a run of N <= 4 (1 KB of LDS each, 256 / D rows).
template <int K, int N, int D>
struct CopyRun {
  static __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, float* lds, int row0,
                                               int sub, int phys, int gstride, int last) {
    constexpr int RPI = 256 / D;
    const int row = row0 + K * RPI + sub;
    const int r = row < last ? row : last;
    const int voff = (r * gstride + ((phys ^ (row & 15)) << 2)) * 4 + 4096 - K * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16,
                                             voff, 0, K * 1024, 0);
    if constexpr (K + 1 < N) CopyRun<K + 1, N, D>::issue(rs, lds, row0, sub, phys, gstride, last);
  }
};

// One wave's share of copying rows 0..R-1 (row r from src + min(r, last) * gstride) into a
// swizzled [R][D] float tile, without staging registers; waited for with wait_vmem_all().
// The buffer starts 4 KB before `src` so that the offsets, which subtract the instruction
// offset, are not negative (only src + row offsets are accessed); R rows x gstride x 4 bytes
// stay below 2^31 for the head counts the C API accepts.
template <int D, int R, int NW>
__device__ __forceinline__ void copy_rows(float* tile, const float* src, int gstride, int last,
                                          int wave, int lane) {
  constexpr int RPI = 256 / D, PER = R / RPI / NW, CPR = D / 4;
  static_assert(PER >= 4 && PER % 4 == 0, "runs of four copy instructions");
  const int sub = lane / CPR, phys = lane % CPR;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(src) - 4096), 0, 0x7fffffff, 0x00020000);
#pragma unroll
  for (int u = 0; u < PER; u += 4) {
    const int u0 = wave * PER + u;
    CopyRun<0, 4, D>::issue(rsrc, tile + u0 * 256, u0 * RPI, sub, phys, gstride, last);
  }
}

// Lane bases (bytes) of the two reads inside a 32-row block of a tile, and the reads.
template <int D>
__device__ __forceinline__ int row_base(int lane) {
  const int c = lane & 31, hh = lane >> 5;
  return c * D * 4 + ((hh ^ (c & 15)) << 4);
}
template <int D>
__device__ __forceinline__ f32x4 row_read(const char* block, int base, int kk) {
  return *reinterpret_cast<const f32x4*>(block + (base ^ (kk << 5)));
}
template <int D>
__device__ __forceinline__ int col_base(int lane) {
  const int c = lane & 31, hh = lane >> 5;
  if constexpr (D == 128) return hh * 4 * D * 4 + ((c ^ (hh * 4)) << 4);
  else return hh * 4 * D * 4 + (((c >> 1) ^ (hh * 4)) << 4) + (c & 1) * 8;
}
template <int D>
__device__ __forceinline__ void col_read(const char* block, int base, int r, float (&x)[D / 32]) {
  const char* p = block + (base ^ ((((r >> 2) & 1) * 8 + (r & 3)) << 4)) +
                  ((r >> 2) * 8 + (r & 3)) * D * 4;
  if constexpr (D == 128) {
    const f32x4 y = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = y[i];
  } else {
    const f32x2 y = *reinterpret_cast<const f32x2*>(p);
    x[0] = y[0];
    x[1] = y[1];
  }
}

// acc += A^T B over the 32 rows of `block`: B (P or dS) in registers, A's columns from LDS.
template <int D>
__device__ __forceinline__ void col_products(const char* block, int cbase, const f32x16& b,
                                             f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float a[D / 32];
    col_read<D>(block, cbase, r, a);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = mfma2(a[db], b[r], acc[db]);
  }
}

// A wave's [32 lanes][D] accumulators (lane c = one query or key) into LDS as swizzled rows.
template <int D>
__device__ __forceinline__ void put_acc(char* block, int lane, const f32x16 (&acc)[D / 32]) {
  const int c = lane & 31, hh = lane >> 5;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = (r >> 2) * 8 + hh * 4 + (r & 3);
    char* row = block + c * D * 4;
    if constexpr (D == 128)
      *reinterpret_cast<f32x4*>(row + ((i ^ (c & 15)) << 4)) =
          f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
    else
      *reinterpret_cast<f32x2*>(row + (((i >> 1) ^ (c & 15)) << 4) + (i & 1) * 8) =
          f32x2{acc[0][r], acc[1][r]};
  }
}
// Chunk ch (head_dim 4 ch ..) of row c of such a block.
template <int D>
__device__ __forceinline__ f32x4 get_chunk(const char* block, int c, int ch) {
  return *reinterpret_cast<const f32x4*>(block + c * D * 4 + ((ch ^ (c & 15)) << 4));
}

constexpr int kThreads = 512, kWaves = 8;  // dK/dV

// Forward and dQ: waves of a workgroup (four for each 32-row query block it holds).  At
// head_dim 64 a workgroup takes one of the two query blocks of a work item, so that two
// workgroups (64 KB of LDS each) run on a CU and small batches spread evenly (both blocks in
// eight waves: dQ 81 against 49 us at the size above); at 128 both (a workgroup's tiles are
// 128 KB of LDS, and four waves would leave the CU with one per SIMD).
template <int D>
__host__ __device__ constexpr int q_waves() { return D == 64 ? 4 : 8; }
template <int D>
inline dim3 q_grid(int64_t n) {
  return dim3((unsigned)(q_waves<D>() == 4 ? (n + 7) / 8 * 16 : n));
}
template <int D>
__device__ __forceinline__ bool query_work(const F32Params& p, WorkItem& it, int& h, int& row0) {
  int b = blockIdx.x;
  row0 = 0;
  if constexpr (q_waves<D>() == 4) {  // the halves of eight blocks' items alternate; the later
    row0 = 32 - ((b >> 3) & 1) * 32;  // rows (more keys) first; b % 8 picks the XCD
    b = (b >> 4) * 8 + (b & 7);
  }
  return block_work(b, p.hdr, p.items, p.hq, p.group, 0, it, h) && row0 < it.a_rows;
}

// Lane's row of a [*, heads, D] tensor as product operands: elements 8 kk + 4 hh .. + 3.
template <int D>
__device__ __forceinline__ void load_frag(f32x4 (&f)[D / 8], const float* row, int hh) {
#pragma unroll
  for (int kk = 0; kk < D / 8; ++kk)
    f[kk] = *reinterpret_cast<const f32x4*>(row + kk * 8 + hh * 4);
}
template <int D>
__device__ __forceinline__ f32x16 row_products(const char* block, int rbase, const f32x4 (&f)[D / 8]) {
  f32x16 s = f32x16{};
#pragma unroll
  for (int kk = 0; kk < D / 8; ++kk) {
    const f32x4 a = row_read<D>(block, rbase, kk);
#pragma unroll
    for (int e = 0; e < 4; ++e) s = mfma2(a[e], f[kk][e], s);
  }
  return s;
}

// Forward.  K and V tiles have one buffer each: V of tile t is copied under the scores of
// tile t, K of tile t+1 under its P V products, a barrier after each half.
template <int D>
__global__ __launch_bounds__(q_waves<D>() * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fwd_f32_kernel(const F32Params p) {
  constexpr int BN = kF32BN, DB = D / 32, NW = q_waves<D>(), QB = NW / 4;
  static_assert(kF32BM == 64 && BN == 128, "tile shape");
  __shared__ __attribute__((aligned(16))) float Kt[BN * D];
  __shared__ __attribute__((aligned(16))) float Vt[BN * D];
  __shared__ float Ms[NW][32], Ls[NW][32];      // per wave and query: max (log2 units), sum
  __shared__ float Wo[QB * 32], Wn[QB * 32];    // running merge: weights of old and new

  WorkItem it;
  int h, row0;  // row0: this workgroup's first row of the item
  if (!query_work<D>(p, it, h, row0)) return;
  const int rows = min(it.a_rows - row0, QB * 32);
  const int hk = h / p.group;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c = lane & 31, hh = lane >> 5;
  const int qb = w & (QB - 1), kb = w / QB;
  const int qrow = qb * 32 + c;
  const int64_t q_start = it.a_start + row0;
  const int64_t qs = (int64_t)p.hq * D;
  const int ks = p.hkv * D;

  f32x4 qf[D / 8];
  load_frag<D>(qf, p.q + (int64_t)(q_start + (qrow < rows ? qrow : 0)) * qs + (int64_t)h * D, hh);
  const float* kbase = p.k + (int64_t)it.b_start * ks + (int64_t)hk * D;
  const float* vbase = p.v + (int64_t)it.b_start * ks + (int64_t)hk * D;
  const int k_len = it.b_len, n_full = it.n0;
  // key tiles that some row of this workgroup sees
  int n_tiles = it.n1;
  if (p.causal && QB == 1)
    n_tiles = min(n_tiles, max(0, it.tile * kF32BM + row0 + rows + it.diag + BN - 1) / BN);
  auto copy = [&](float* dst, const float* src, int t) {
    copy_rows<D, BN, NW>(dst, src + (int64_t)t * BN * ks, ks, k_len - 1 - t * BN, w, lane);
  };

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
  float m2 = -INFINITY, l_run = 0.f;
  const float c2 = p.scale_log2;
  const int q_rel = it.tile * kF32BM + row0 + qrow;
  int lim_base = k_len;  // keys below it are visible to this lane's query
  if (p.causal) lim_base = min(k_len, q_rel + it.diag + 1);
  lim_base -= hh * 4;
  // keys below it are visible to some query of this wave
  int wave_lim = k_len;
  if (p.causal) wave_lim = min(k_len, it.tile * kF32BM + row0 + min(qb * 32 + 32, rows) + it.diag);
  if (qb * 32 >= rows) wave_lim = 0;
  const char* kblk = reinterpret_cast<const char*>(Kt + kb * 32 * D);
  const char* vblk = reinterpret_cast<const char*>(Vt + kb * 32 * D);
  const int rbase = row_base<D>(lane), cbase = col_base<D>(lane);

  if (n_tiles > 0) copy(Kt, kbase, 0);
  wait_vmem_all();
  __syncthreads();
  for (int t = 0; t < n_tiles; ++t) {
    copy(Vt, vbase, t);
    const int k0 = t * BN + kb * 32;
    const bool live = k0 < wave_lim;
    f32x16 s = f32x16{};
    if (live) s = row_products<D>(kblk, rbase, qf);
    wait_vmem_all();
    __syncthreads();  // V of tile t has landed; every wave is done with K
    if (t + 1 < n_tiles) copy(Kt, kbase, t + 1);
    if (live) {
      if (t >= n_full) {
        const int lim = lim_base - k0;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = ((r >> 2) * 8 + (r & 3)) < lim ? s[r] : -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
      mx = half_max(mx) * c2;
      if (__any(mx > m2)) {
        const float m_new = fmaxf(m2, mx);
        const float alpha = fast_exp2(m2 - (m_new == -INFINITY ? 0.f : m_new));
        m2 = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
      }
      const float base = m2 == -INFINITY ? 0.f : m2;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = fast_exp2(fmaf(s[r], c2, -base));
        l_run += s[r];
      }
      col_products<D>(vblk, cbase, s, oacc);
    }
    wait_vmem_all();
    __syncthreads();  // K of tile t+1 has landed; every wave is done with V
  }

  // combine the four key blocks' (max, sum, O) of each query
  const float l_tot = half_sum(l_run);
  if (hh == 0) {
    Ms[w][c] = m2;
    Ls[w][c] = l_tot;
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) M = fmaxf(M, Ms[i * QB + qb][c]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float mi = Ms[i * QB + qb][c];
    L += Ls[i * QB + qb][c] * (mi == -INFINITY ? 0.f : fast_exp2(mi - M));
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;
  const float wgt = m2 == -INFINITY ? 0.f : fast_exp2(m2 - M) * inv;
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] *= wgt;
  auto area = [&](int wv) {
    return reinterpret_cast<char*>(wv < NW / 2 ? Kt : Vt) + (wv % (NW / 2)) * 32 * D * 4;
  };
  put_acc<D>(area(w), lane, oacc);
  if (kb == 0 && hh == 0 && qrow < rows) {
    const int64_t row = q_start + qrow;
    const float lse2 = L > 0.f ? M + log2f(L) : -INFINITY;  // log2 domain
    if (p.o_run == nullptr) {
      p.lse_out[(int64_t)h * p.total_q + row] = lse2 * kLn2;
    } else {  // log-sum-exp weights of the running state and of this step
      float* lr = p.lse_run + (int64_t)h * p.total_q + row;
      const float old2 = p.accumulate ? *lr * kLog2e : -INFINITY;
      const float mx = fmaxf(old2, lse2);
      float w_old = 0.f, w_new = 0.f, lse_m = -INFINITY;
      if (mx != -INFINITY) {
        const float eo = fast_exp2(old2 - mx), en = fast_exp2(lse2 - mx);
        w_old = eo / (eo + en);
        w_new = en / (eo + en);
        lse_m = (mx + log2f(eo + en)) * kLn2;
      }
      Wo[qrow] = w_old;
      Wn[qrow] = w_new;
      *lr = lse_m;
    }
  }
  __syncthreads();
  for (int u = tid; u < QB * 32 * (D / 4); u += NW * 64) {
    const int r = u / (D / 4), ch = u % (D / 4);
    if (r >= rows) break;  // rows come in order
    f32x4 x = get_chunk<D>(area(r >> 5), r & 31, ch);
#pragma unroll
    for (int i = 1; i < 4; ++i) x += get_chunk<D>(area(i * QB + (r >> 5)), r & 31, ch);
    const int64_t off = (int64_t)(q_start + r) * qs + (int64_t)h * D + ch * 4;
    if (p.o_run == nullptr) {
      *reinterpret_cast<f32x4*>(p.o + off) = x;
    } else {
      x *= Wn[r];
      if (Wo[r] != 0.f) x += *reinterpret_cast<const f32x4*>(p.o_run + off) * Wo[r];
      *reinterpret_cast<f32x4*>((p.o != nullptr ? p.o : p.o_run) + off) = x;
    }
  }
}

// dQ: sum over visible keys of dS_ij k_j, dS = P (dO.v_j - D); forms D = rowsum(dO * O) too.
// V of tile t+1 is copied under the dQ products of tile t, K after them.
template <int D>
__global__ __launch_bounds__(q_waves<D>() * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dq_f32_kernel(const F32Params p) {
  constexpr int BN = kF32BN, DB = D / 32, NW = q_waves<D>(), QB = NW / 4;
  __shared__ __attribute__((aligned(16))) float Kt[BN * D];
  __shared__ __attribute__((aligned(16))) float Vt[BN * D];

  WorkItem it;
  int h, row0;  // row0: this workgroup's first row of the item
  if (!query_work<D>(p, it, h, row0)) return;
  const int rows = min(it.a_rows - row0, QB * 32);
  const int hk = h / p.group;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c = lane & 31, hh = lane >> 5;
  const int qb = w & (QB - 1), kb = w / QB;
  const int qrow = qb * 32 + c;
  const bool qvalid = qrow < rows;
  const int64_t q_start = it.a_start + row0;
  const int64_t qs = (int64_t)p.hq * D;
  const int ks = p.hkv * D;
  const int64_t qoff = (int64_t)(q_start + (qvalid ? qrow : 0)) * qs + (int64_t)h * D;

  f32x4 qf[D / 8], dof[D / 8];
  load_frag<D>(qf, p.q + qoff, hh);
  load_frag<D>(dof, p.dout + qoff, hh);
  float dpart = 0.f;
#pragma unroll
  for (int kk = 0; kk < D / 8; ++kk) {
    const f32x4 ov = *reinterpret_cast<const f32x4*>(p.out + qoff + kk * 8 + hh * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) dpart = fmaf(dof[kk][e], ov[e], dpart);
  }
  const float drow = half_sum(dpart);
  float lse2 = INFINITY, dval = 0.f;
  if (qvalid) {
    const int64_t ri = (int64_t)h * p.total_q + q_start + qrow;
    const float l = p.lse[ri];
    lse2 = l == -INFINITY ? INFINITY : l * kLog2e;
    dval = drow;
    if (kb == 0 && hh == 0) p.dvec[ri] = drow;
  }
  const float* kbase = p.k + (int64_t)it.b_start * ks + (int64_t)hk * D;
  const float* vbase = p.v + (int64_t)it.b_start * ks + (int64_t)hk * D;
  const int k_len = it.b_len, n_full = it.n0;
  // key tiles that some row of this workgroup sees
  int n_tiles = it.n1;
  if (p.causal && QB == 1)
    n_tiles = min(n_tiles, max(0, it.tile * kF32BM + row0 + rows + it.diag + BN - 1) / BN);
  auto copy = [&](float* dst, const float* src, int t) {
    copy_rows<D, BN, NW>(dst, src + (int64_t)t * BN * ks, ks, k_len - 1 - t * BN, w, lane);
  };
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
  const int q_rel = it.tile * kF32BM + row0 + qrow;
  int lim_base = k_len;
  if (p.causal) lim_base = min(k_len, q_rel + it.diag + 1);
  lim_base -= hh * 4;
  int wave_lim = k_len;
  if (p.causal) wave_lim = min(k_len, it.tile * kF32BM + row0 + min(qb * 32 + 32, rows) + it.diag);
  if (qb * 32 >= rows) wave_lim = 0;
  const char* kblk = reinterpret_cast<const char*>(Kt + kb * 32 * D);
  const char* vblk = reinterpret_cast<const char*>(Vt + kb * 32 * D);
  const int rbase = row_base<D>(lane), cbase = col_base<D>(lane);

  if (n_tiles > 0) {
    copy(Kt, kbase, 0);
    copy(Vt, vbase, 0);
  }
  wait_vmem_all();
  __syncthreads();
  for (int t = 0; t < n_tiles; ++t) {
    const int k0 = t * BN + kb * 32;
    const bool live = k0 < wave_lim;
    f32x16 s = f32x16{}, dp = f32x16{};
    if (live) {
      s = row_products<D>(kblk, rbase, qf);
      dp = row_products<D>(vblk, rbase, dof);
    }
    __syncthreads();  // every wave is done with V
    if (t + 1 < n_tiles) copy(Vt, vbase, t + 1);
    if (live) {
      if (t >= n_full) {
        const int lim = lim_base - k0;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = ((r >> 2) * 8 + (r & 3)) < lim ? s[r] : -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
        s[r] = fast_exp2(fmaf(s[r], p.scale_log2, -lse2)) * (dp[r] - dval);
      col_products<D>(kblk, cbase, s, acc);
    }
    __syncthreads();  // every wave is done with K
    if (t + 1 < n_tiles) {
      copy(Kt, kbase, t + 1);
      wait_vmem_all();
      __syncthreads();
    }
  }
  auto area = [&](int wv) {
    return reinterpret_cast<char*>(wv < NW / 2 ? Kt : Vt) + (wv % (NW / 2)) * 32 * D * 4;
  };
  put_acc<D>(area(w), lane, acc);
  __syncthreads();
  for (int u = tid; u < QB * 32 * (D / 4); u += NW * 64) {
    const int r = u / (D / 4), ch = u % (D / 4);
    if (r >= rows) break;
    f32x4 x = get_chunk<D>(area(r >> 5), r & 31, ch);
#pragma unroll
    for (int i = 1; i < 4; ++i) x += get_chunk<D>(area(i * QB + (r >> 5)), r & 31, ch);
    x *= p.scale;
    f32x4* dst = reinterpret_cast<f32x4*>(p.dq + (int64_t)(q_start + r) * qs + (int64_t)h * D + ch * 4);
    if (p.dq_accumulate) x += *dst;
    *dst = x;
  }
}

// dK, dV of 32 keys, summed over the query heads of their group.  Wave (qb, role): S waves
// (role 0, K of the keys in registers) form S, P and dV, dP waves (role 1, V) dP, dS and dK
// for the 32-row block qb of each query tile; P goes from one to the other through LDS.  At
// head_dim 64 the tiles are double-buffered; at 128 two tiles fill the LDS.
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dkdv_f32_kernel(const F32Params p) {
  constexpr int BM = kF32BwdBM, BN = kF32BwdBN, DB = D / 32;
  constexpr bool kDouble = D == 64;
  static_assert(BM == 128 && BN == 32, "tile shape");
  __shared__ __attribute__((aligned(16))) float Q0[BM * D];
  __shared__ __attribute__((aligned(16))) float dO0[BM * D];
  __shared__ __attribute__((aligned(16))) float Q1[kDouble ? BM * D : 4];
  __shared__ __attribute__((aligned(16))) float dO1[kDouble ? BM * D : 4];
  __shared__ __attribute__((aligned(16))) f32x4 Ps[4][4][64];  // [query block][quad][lane]

  WorkItem it;
  int hk;
  const int slab = blockIdx.x % p.splits;
  if (!block_work(blockIdx.x / p.splits, p.hdr, p.items, p.hkv, 1, kHeadMajorRowsDkdv, it, hk)) return;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c = lane & 31, hh = lane >> 5;
  const int qb = w & 3, role = w >> 2;
  const int64_t qs = (int64_t)p.hq * D, ks = (int64_t)p.hkv * D;
  const int key_rel = it.tile * BN + c;

  f32x4 frag[D / 8];
  load_frag<D>(frag, (role == 0 ? p.k : p.v) +
                         (int64_t)(it.a_start + (c < it.a_rows ? c : 0)) * ks + (int64_t)hk * D, hh);
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
  const int q_len = it.b_len, n_vis = it.n2;
  // this workgroup's steps
  const int i_first = slab * (n_vis * p.group) / p.splits;
  const int n_iter = (slab + 1) * (n_vis * p.group) / p.splits;
  const int rbase = row_base<D>(lane), cbase = col_base<D>(lane);

  // tile i into (Qd, dOd), and lane c's row of this wave's block: its LSE or D
  float row_raw = 0.f;
  bool row_ok = false;
  auto copy = [&](int i, float* Qd, float* dOd) {
    const int hg = i / n_vis, j = i - hg * n_vis;
    const int h = hk * p.group + hg;
    const int q_rel0 = (it.n0 + j) * BM;
    const int64_t q_glob0 = (int64_t)it.b_start + q_rel0;
    const int last = q_len - 1 - q_rel0;
    const int64_t qo = q_glob0 * qs + (int64_t)h * D;
    copy_rows<D, BM, kWaves>(Qd, p.q + qo, (int)qs, last, w, lane);
    copy_rows<D, BM, kWaves>(dOd, p.dout + qo, (int)qs, last, w, lane);
    row_ok = qb * 32 + c <= last;
    row_raw = (role == 0 ? p.lse : p.dvec)[(int64_t)h * p.total_q + q_glob0 +
                                          (row_ok ? qb * 32 + c : 0)];
  };
  if (n_iter > i_first) copy(i_first, Q0, dO0);
  wait_vmem_all();
  __syncthreads();

  auto step = [&](int i, const float* Qb, const float* dOb, float* Qn, float* dOn) {
    const int j = i % n_vis;
    const int q_rel0 = (it.n0 + j) * BM;
    // LSE in log2 units, +inf (P = 0) past the segment and where no key is visible; or D
    const float rowv = role == 0 ? ((!row_ok || row_raw == -INFINITY) ? INFINITY : row_raw * kLog2e)
                                 : (row_ok ? row_raw : 0.f);
    if (kDouble && i + 1 < n_iter) copy(i + 1, Qn, dOn);
    const char* rblk = reinterpret_cast<const char*>((role == 0 ? Qb : dOb) + qb * 32 * D);
    const char* cblk = reinterpret_cast<const char*>((role == 0 ? dOb : Qb) + qb * 32 * D);
    // rows of this block exist and, on MASKED tiles of a causal pass, its last row sees the
    // tile's first key
    const bool masked = j < it.n1 && p.causal;
    const int row0 = q_rel0 + qb * 32;
    const bool live = row0 < q_len && (!masked || it.tile * BN - (row0 + 31) <= it.diag);
    f32x16 s = f32x16{};
    if (live) {
      s = row_products<D>(rblk, rbase, frag);
      if (role == 0) {
        const int vis_lim = key_rel - it.diag - row0 - hh * 4;  // rows below it are hidden
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lse2 = __shfl(rowv, a4 * 8 + hh * 4 + e);
            float pr = fast_exp2(fmaf(s[a4 * 4 + e], p.scale_log2, -lse2));
            if (masked) pr = (a4 * 8 + e) >= vis_lim ? pr : 0.f;
            s[a4 * 4 + e] = pr;
          }
          Ps[qb][a4][lane] = f32x4{s[a4 * 4], s[a4 * 4 + 1], s[a4 * 4 + 2], s[a4 * 4 + 3]};
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] -= __shfl(rowv, (r >> 2) * 8 + hh * 4 + (r & 3));
      }
    }
    barrier_lds();  // P is in LDS (the copies of tile i+1 stay in flight)
    if (live) {
      if (role == 1) {
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
          const f32x4 p4 = Ps[qb][a4][lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) s[a4 * 4 + e] *= p4[e];
        }
      }
      col_products<D>(cblk, cbase, s, acc);
    }
    wait_vmem_all();
    __syncthreads();
    if (!kDouble && i + 1 < n_iter) {
      copy(i + 1, Qn, dOn);
      wait_vmem_all();
      __syncthreads();
    }
  };
  if constexpr (kDouble) {
    for (int i = i_first; i < n_iter; i += 2) {
      step(i, Q0, dO0, Q1, dO1);
      if (i + 1 < n_iter) step(i + 1, Q1, dO1, Q0, dO0);
    }
  } else {
    for (int i = i_first; i < n_iter; ++i) step(i, Q0, dO0, Q0, dO0);
  }
  auto area = [&](int b, int rl) {
    return reinterpret_cast<char*>(rl == 0 ? Q0 : dO0) + b * 32 * D * 4;
  };
  put_acc<D>(area(qb, role), lane, acc);
  __syncthreads();
  for (int u = tid; u < 2 * BN * (D / 4); u += kThreads) {
    const int rl = u / (BN * (D / 4)), r = u / (D / 4) % BN, ch = u % (D / 4);
    if (r >= it.a_rows) continue;
    f32x4 x = get_chunk<D>(area(0, rl), r, ch);
#pragma unroll
    for (int b = 1; b < 4; ++b) x += get_chunk<D>(area(b, rl), r, ch);
    if (rl == 1) x *= p.scale;
    const int64_t off = (int64_t)(it.a_start + r) * ks + (int64_t)hk * D + ch * 4;
    if (p.splits > 1) {  // dV's slabs come behind dK's
      *reinterpret_cast<f32x4*>(p.part + ((1 - rl) * p.splits + slab) * p.total_k * ks + off) = x;
      continue;
    }
    f32x4* dst = reinterpret_cast<f32x4*>((rl == 0 ? p.dv : p.dk) + off);
    if (p.kv_accumulate) x += *dst;
    *dst = x;
  }
}

F32Params make_params(const bs_dims& dims, const void* q, const void* k, const void* v,
                      const void* ws, const WsLayout& L, int causal, float scale) {
  F32Params p = {};
  p.q = static_cast<const float*>(q);
  p.k = static_cast<const float*>(k);
  p.v = static_cast<const float*>(v);
  p.hdr = static_cast<const WsHeader*>(ws);
  p.items = reinterpret_cast<const WorkItem*>(static_cast<const char*>(ws) + L.sorted);
  p.total_q = dims.total_q;
  p.hq = dims.hq;
  p.hkv = dims.hkv;
  p.group = dims.hq / dims.hkv;
  p.causal = causal;
  p.scale = scale;
  p.scale_log2 = scale * kLog2e;
  return p;
}

}  // namespace

hipError_t launch_fwd_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                          int causal, float scale, void* out, float* lse, const FwdMerge* merge,
                          const void* ws, const WsLayout& L, hipStream_t stream) {
  if (L.max_items == 0 || dims.hq == 0) return hipSuccess;
  F32Params p = make_params(dims, q, k, v, ws, L, causal, scale);
  p.o = static_cast<float*>(out);
  p.lse_out = lse;
  p.o_run = merge ? merge->o_run : nullptr;
  p.lse_run = merge ? merge->lse_run : nullptr;
  p.accumulate = merge ? merge->accumulate : 0;
  const int64_t n = L.max_items * dims.hq;
  if (dims.head_dim == 128)
    hipLaunchKernelGGL(fwd_f32_kernel<128>, q_grid<128>(n), dim3(q_waves<128>() * 64), 0, stream, p);
  else
    hipLaunchKernelGGL(fwd_f32_kernel<64>, q_grid<64>(n), dim3(q_waves<64>() * 64), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_dq_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                         const void* out, const void* dout, const float* lse, float* dvec,
                         int causal, float scale, void* dq, int dq_accumulate, const void* ws,
                         const WsLayout& L, hipStream_t stream) {
  if (L.max_items == 0 || dims.hq == 0) return hipSuccess;
  F32Params p = make_params(dims, q, k, v, ws, L, causal, scale);
  p.out = static_cast<const float*>(out);
  p.dout = static_cast<const float*>(dout);
  p.lse = lse;
  p.dvec = dvec;
  p.dq = static_cast<float*>(dq);
  p.dq_accumulate = dq_accumulate;
  const int64_t n = L.max_items * dims.hq;
  if (dims.head_dim == 128)
    hipLaunchKernelGGL(dq_f32_kernel<128>, q_grid<128>(n), dim3(q_waves<128>() * 64), 0, stream, p);
  else
    hipLaunchKernelGGL(dq_f32_kernel<64>, q_grid<64>(n), dim3(q_waves<64>() * 64), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_dkdv_f32(const bs_dims& dims, const void* q, const void* k, const void* v,
                           const void* dout, const float* lse, const float* dvec, int causal,
                           float scale, void* dk, void* dv, int kv_accumulate, const void* ws,
                           const WsLayout& L, int splits, float* part, hipStream_t stream) {
  if (L.max_items == 0 || dims.hkv == 0) return hipSuccess;
  F32Params p = make_params(dims, q, k, v, ws, L, causal, scale);
  p.kv_accumulate = kv_accumulate;
  p.splits = splits;
  p.part = part;
  p.total_k = dims.total_k;
  p.dout = static_cast<const float*>(dout);
  p.lse = lse;
  p.dvec = const_cast<float*>(dvec);
  p.dk = static_cast<float*>(dk);
  p.dv = static_cast<float*>(dv);
  const dim3 grid((unsigned)(L.max_items * dims.hkv * splits));
  if (dims.head_dim == 128) hipLaunchKernelGGL(dkdv_f32_kernel<128>, grid, dim3(kThreads), 0, stream, p);
  else hipLaunchKernelGGL(dkdv_f32_kernel<64>, grid, dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace bs
