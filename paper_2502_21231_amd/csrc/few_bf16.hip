// bf16 attention forward for segments of few queries over many keys (decoding, the last tokens
// of a cached prompt), gfx950.
//
// Such a call is bound by reading K and V once (2 x 2 x head_dim bytes per key and KV head; a
// 32-row product tile needs a twentieth of that time), so the kernel is laid out for memory:
//   - the query heads of a KV group are rows of one 32-row product block, row qi * group + hg
//     of segment b being query qi of head hk * group + hg, so the group reads its K and V once
//     (the general kernel, one head and 128 rows per workgroup, reads them once per head);
//   - the keys of all segments, in blocks of 4 x KT keys, form one line per KV head that is cut
//     into as many equal ranges as there are workgroups (two per CU), whatever the lengths: a
//     workgroup's range may begin and end inside a segment.  A piece of a segment that does not
//     hold all of it leaves its (O, max, sum) in float32 in the workspace, and few_merge_kernel
//     combines the pieces of each row;
//   - the four waves of a workgroup take the block's KT-key tiles in turn, each with an LDS
//     buffer of its own (8 KB of K, 8 KB of V) that it fills (buffer_load ... lds) and waits for
//     by itself: no workgroup barrier per tile, and eight waves keep up to 128 KB per CU in
//     flight.  The next K is requested as soon as the scores are done with this one.
// Measured (both launches): 32 sequences of one query over up to 8K keys, 64/8 heads, head_dim
// 128 (394 MB of keys): 336 -> 76 us, 5.2 TB/s (a plain device copy moves 4.9); one sequence over
// 16K keys: 90 -> 20 us; 16 x 8 queries, 32/32 heads: 110 -> 79 us.  Non-temporal copies (keys
// read once): 88 -> 76 us at the first size, but 61 -> 67 us where four row blocks read them.
// There is no separate plan: every workgroup validates cu_seqlens and lays out the line from
// them (up to kFewMaxSegs segments), which costs about as much as reading a work list.
// Orientation, swizzled tiles and softmax are those of fwd_bf16.hip.
#include <type_traits>

#include "attn.hpp"

namespace bs {
namespace {

struct FewParams {
  const bf16* q;
  const bf16* k;
  const bf16* v;
  bf16* o;
  float* lse;
  const int32_t* cu_q;
  const int32_t* cu_k;
  WsHeader* hdr;
  float* part;   // [slabs][total_q * hq][D] sums of the pieces
  float2* stat;  // [slabs][total_q * hq] (max in log2 units, sum)
  int32_t* cnt;  // [total_q * hq] pieces of the row
  int64_t total_q, total_k;
  int32_t num_seqs, max_seqlen;
  int32_t hq, hkv, group;
  int32_t causal;
  int32_t slabs;    // pieces of a row at most
  int32_t per_min;  // blocks per workgroup that keep to it with a segment of max_seqlen keys
  float scale_log2;
};

// Waits until at most N of this wave's copies are under way (a builtin, so that the compiler
// knows and adds no wait of its own; the clobbers keep LDS accesses on their side of it).
template <int N>
__device__ __forceinline__ void wait_copies() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | N);  // vmcnt(N), N < 16
  asm volatile("" ::: "memory");
}
// This wave's LDS reads have returned: their buffer may be copied into.
__device__ __forceinline__ void wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int D, int kAux>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void few_fwd_kernel(const FewParams p) {
  constexpr int KT = D == 128 ? 32 : 64;  // keys of a wave's tile
  constexpr int KB = KT / 32, KK = D / 16, DB = D / 32;
  constexpr int BLK = 4 * KT;
  __shared__ __attribute__((aligned(16))) bf16 Kt[4][KT * D];
  __shared__ __attribute__((aligned(16))) bf16 Vt[4][KT * D];
  __shared__ int32_t pre[kFewMaxSegs + 1];  // blocks before each segment, per KV head
  __shared__ int32_t wsum[4];
  __shared__ int32_t bad;
  __shared__ float Ms[4][32], Ls[4][32];

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c = lane & 31, hh = lane >> 5;
  const int group = p.group;

  // the line of blocks: thread t takes segments 4t .. 4t+3
  if (tid == 0) bad = 0;
  __syncthreads();
  {
    if (tid == 0) {
      int code = 0;
      if (p.cu_q[p.num_seqs] != p.total_q || p.cu_k[p.num_seqs] != p.total_k) code = BS_DEV_BAD_TOTAL;
      if (p.cu_q[0] != 0 || p.cu_k[0] != 0) code = BS_DEV_BAD_FIRST;
      if (code != 0) atomicCAS(&bad, 0, code);
    }
    constexpr int PT = kFewMaxSegs / 256;
    int32_t n[PT], sum = 0;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int b = tid * PT + i;
      n[i] = 0;
      if (b < p.num_seqs) {
        const int64_t lq = (int64_t)p.cu_q[b + 1] - p.cu_q[b], lk = (int64_t)p.cu_k[b + 1] - p.cu_k[b];
        if (lq < 0 || lk < 0) atomicCAS(&bad, 0, BS_DEV_NOT_MONOTONE);
        else if (lq > p.max_seqlen || lk > p.max_seqlen) atomicCAS(&bad, 0, BS_DEV_TOO_LONG);
        else if (lq > 0) n[i] = (int32_t)((lq * group + 31) / 32 * max((lk + BLK - 1) / BLK, (int64_t)1));
      }
      sum += n[i];
    }
    int32_t run = sum;  // inclusive scan over the wave, then over the four waves
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t x = __shfl_up(run, off);
      if (lane >= off) run += x;
    }
    if (lane == 63) wsum[w] = run;
    __syncthreads();
    int32_t at = run - sum;
    for (int i = 0; i < w; ++i) at += wsum[i];
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int b = tid * PT + i;
      if (b <= p.num_seqs) pre[b] = at;
      at += n[i];
    }
    if (tid == 255 && p.num_seqs == kFewMaxSegs) pre[kFewMaxSegs] = at;
    __syncthreads();
  }
  const int code = bad;
  if (blockIdx.x == 0 && tid == 0) {
    p.hdr->status = code;
    p.hdr->n_items = 0;
  }
  if (code != 0) return;  // uniform: nothing is written
  const int32_t line = pre[p.num_seqs];
  const int64_t all = (int64_t)line * p.hkv;
  int32_t per = (int32_t)((all + gridDim.x - 1) / gridDim.x);
  if (per < p.per_min) {  // uniform
    // by the longest segment, since max_seqlen is only a bound (67 sequences of 1 to 20 queries over up
    // to 651 keys, 32/8 heads, max_seqlen 26K: 100 us by the bound, 34 so)
    int32_t most = 0;
    for (int b = tid; b < p.num_seqs; b += 256)
      if (p.cu_q[b + 1] > p.cu_q[b]) most = max(most, (p.cu_k[b + 1] - p.cu_k[b] + BLK - 1) / BLK);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) most = max(most, __shfl_xor(most, off));
    if (lane == 0) wsum[w] = most;
    __syncthreads();
    per = max(per, few_per_min(max(max(wsum[0], wsum[1]), max(wsum[2], wsum[3])), p.slabs));
  }
  int64_t x = (int64_t)blockIdx.x * per;
  const int64_t x_end = min(all, x + per);

  bf16* Kw = Kt[w];
  bf16* Vw = Vt[w];
  const int rbase = swz_row_base<D>(lane), tbase = swz_tr_base<D>(lane);
  const int64_t qstride = (int64_t)p.hq * D;
  const int kvstride = p.hkv * D;
  const int64_t all_rows = p.total_q * p.hq;

  while (x < x_end) {
    // the piece that starts at x: KV head, segment, row block, key blocks [kb0, kb0 + n)
    const int hk = (int)(x / line);
    const int32_t y = (int32_t)(x - (int64_t)hk * line);
    int lo = 0, hi = p.num_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (pre[mid] <= y) lo = mid; else hi = mid - 1;
    }
    const int64_t q_start = p.cu_q[lo], k_start = p.cu_k[lo];
    const int lq = p.cu_q[lo + 1] - (int)q_start, lk = p.cu_k[lo + 1] - (int)k_start;
    const int nkb = max((lk + BLK - 1) / BLK, 1);
    const int rb = (y - pre[lo]) / nkb, kb0 = (y - pre[lo]) - rb * nkb;
    const int n = (int)min((int64_t)(nkb - kb0), x_end - x);
    const int64_t xs = (int64_t)hk * line + pre[lo] + (int64_t)rb * nkb;  // the row block's first
    const int slab = (int)(blockIdx.x - xs / per);
    const int pieces = (int)((xs + nkb - 1) / per - xs / per) + 1;
    x += n;

    const int rows = min(lq * group - rb * 32, 32);
    const int r_lane = rb * 32 + min(c, rows - 1);
    const int qi = r_lane / group, hg = r_lane - qi * group;
    bf16x8 qf[KK];
    {
      const bf16* qp = p.q + (q_start + qi) * qstride + (int64_t)(hk * group + hg) * D + hh * 8;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
    }
    const bf16* kbase = p.k + k_start * kvstride + (int64_t)hk * D;
    const bf16* vbase = p.v + k_start * kvstride + (int64_t)hk * D;
    const int diag = lk - lq;
    const int lim_lane = (p.causal ? min(lk, qi + diag + 1) : lk) - hh * 4;
    // keys some row of the block sees, and this piece's end
    int k_end = min(lk, (kb0 + n) * BLK);
    if (p.causal) k_end = min(k_end, (rb * 32 + rows - 1) / group + diag + 1);

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
    float m2 = -INFINITY, l_run = 0.f;
    const float c2 = p.scale_log2;

    int k0 = (kb0 * 4 + w) * KT;
    // the copies of a tile: 8 instructions each for K and V
    auto copy = [&](bf16* dst, const bf16* src, int key) {
      const bf16* s = src + (int64_t)key * kvstride;
      const int last = lk - 1 - key;
#pragma unroll
      for (int half = 0; half < 2; ++half) dma_tile<D, KT, 2, kAux>(dst, s, kvstride, last, half, lane);
    };
    // one tile; `more`: another follows (two straight-line forms: behind a branch the compiler
    // would lose count of the copies and wait for all of them)
    auto step = [&](auto more) {
      wait_copies<8>();  // K has landed (V's eight copies may be under way)
      f32x16 s[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) s[kb] = f32x16{};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const bf16x8 a = lds_row16(Kw, (rbase ^ (kk << 5)) + kb * 64 * D);
          s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], s[kb], 0, 0, 0);
        }
      const int next = k0 + BLK;
      wait_reads();
      if constexpr (more()) copy(Kw, kbase, next);
      const int lim = lim_lane - k0;
      if (k0 + KT > lk || p.causal) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            s[kb][r] = (kb * 32 + (r >> 2) * 8 + (r & 3)) < lim ? s[kb][r] : -INFINITY;
      }
      float mx = s[0][0];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
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
      bf16x8 pb[2 * KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float e = fast_exp2(fmaf(s[kb][r], c2, -base));
          l_run += e;
          pb[kb * 2 + (r >> 3)][r & 7] = f2bf(e);
        }
      wait_copies<more() ? 8 : 0>();  // V has landed
#pragma unroll
      for (int ks = 0; ks < 2 * KB; ++ks)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const bf16x8 a = lds_tr16(Vw, (tbase ^ (db << 6)) + ks * 32 * D,
                                    (tbase ^ ((db << 6) | 32)) + ks * 32 * D + 16 * D);
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[ks], oacc[db], 0, 0, 0);
        }
      wait_reads();
      if constexpr (more()) copy(Vw, vbase, next);
      k0 = next;
    };

    if (k0 < k_end) {
      copy(Kw, kbase, k0);
      copy(Vw, vbase, k0);
      // Q is waited for here: left to the loop, the compiler would wait for every copy there
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qf[kk]));
      while (k0 + BLK < k_end) step(std::true_type{});
      step(std::false_type{});
    }

    // combine the four waves' (max, sum, O): O in the wave's own buffers, head_dim in two halves
    // of 64 columns at head_dim 128, 16-byte chunk k of row c at chunk k ^ (c & 15)
    const float l_tot = half_sum(l_run);
    if (hh == 0) {
      Ms[w][c] = m2;
      Ls[w][c] = l_tot;
    }
    __syncthreads();
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) M = fmaxf(M, Ms[i][c]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float mi = Ms[i][c];
      L += Ls[i][c] * (mi == -INFINITY ? 0.f : fast_exp2(mi - M));
    }
    const bool whole = pieces == 1;
    float wgt = m2 == -INFINITY ? 0.f : fast_exp2(m2 - M);
    if (whole) wgt *= L > 0.f ? 1.f / L : 0.f;
    auto area = [&](int wv, int ch) {  // chunk ch (head_dim 4 ch ..) of row 0
      return reinterpret_cast<char*>(ch < 16 ? Kt[wv] : Vt[wv]);
    };
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int ch = db * 8 + a * 2 + hh;
        const f32x4 o4 = {oacc[db][a * 4] * wgt, oacc[db][a * 4 + 1] * wgt,
                          oacc[db][a * 4 + 2] * wgt, oacc[db][a * 4 + 3] * wgt};
        *reinterpret_cast<f32x4*>(area(w, db * 8) + c * 256 + (((ch & 15) ^ (c & 15)) << 4)) = o4;
      }
    if (w == 0 && hh == 0 && c < rows) {
      const int h = hk * group + hg;
      const int64_t row = (q_start + qi) * p.hq + h;
      if (whole) p.lse[(int64_t)h * p.total_q + q_start + qi] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
      else p.stat[(int64_t)slab * all_rows + row] = make_float2(M, L);
      if (slab == 0 && p.cnt != nullptr) p.cnt[row] = pieces;
    }
    __syncthreads();
    for (int u = tid; u < rows * (D / 4); u += 256) {
      const int r = u / (D / 4), ch = u % (D / 4);
      const int at = r * 256 + (((ch & 15) ^ (r & 15)) << 4);
      f32x4 o4 = *reinterpret_cast<const f32x4*>(area(0, ch) + at);
#pragma unroll
      for (int i = 1; i < 4; ++i) o4 += *reinterpret_cast<const f32x4*>(area(i, ch) + at);
      const int rr = rb * 32 + r, ri = rr / group;
      const int64_t row = (q_start + ri) * p.hq + hk * group + (rr - ri * group);
      if (whole)
        *reinterpret_cast<bf16x4*>(p.o + row * D + ch * 4) =
            bf16x4{f2bf(o4[0]), f2bf(o4[1]), f2bf(o4[2]), f2bf(o4[3])};
      else
        *reinterpret_cast<f32x4*>(p.part + ((int64_t)slab * all_rows + row) * D + ch * 4) = o4;
    }
    __syncthreads();  // the buffers are free
  }
}

// Rows in several pieces: O = sum 2^(M_i - M) O_i / L, LSE = (M + log2 L) ln 2,
// L = sum 2^(M_i - M) L_i.  D/4 lanes per row, 16 bytes each; each lane weighs pieces ch and
// ch + D/4, so that no lane waits for the pieces one after another.
template <int D>
__global__ __launch_bounds__(256) void few_merge_kernel(const FewParams p) {
  if (p.hdr->status != BS_DEV_OK) return;
  constexpr int LPR = D / 4, NP = kFewSlabs / LPR;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = gid / LPR, rows = p.total_q * p.hq;
  const int ch = (int)(gid % LPR), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int n = p.cnt[row];
  if (n <= 1) return;
  float m[NP], wgt[NP], M = -INFINITY, L = 0.f;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int i = ch + j * LPR;
    const float2 st = i < n ? p.stat[i * rows + row] : make_float2(-INFINITY, 0.f);
    m[j] = st.x;
    wgt[j] = st.y;
    M = fmaxf(M, m[j]);
  }
#pragma unroll
  for (int off = 1; off < LPR; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
  const float base = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    m[j] = fast_exp2(m[j] - base);
    L += wgt[j] * m[j];
  }
#pragma unroll
  for (int off = 1; off < LPR; off <<= 1) L += __shfl_xor(L, off);
  f32x4 o = f32x4{};
  const float* src = p.part + row * D + ch * 4;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int nj = min(LPR, n - j * LPR);
#pragma unroll 8
    for (int i = 0; i < nj; ++i)
      o += *reinterpret_cast<const f32x4*>(src + (int64_t)(i + j * LPR) * rows * D) *
           __shfl(m[j], (lane & ~(LPR - 1)) + i);
  }
  o *= L > 0.f ? 1.f / L : 0.f;
  *reinterpret_cast<bf16x4*>(p.o + row * D + ch * 4) =
      bf16x4{f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3])};
  if (ch == 0) {
    const int64_t t = row / p.hq;
    p.lse[(row - t * p.hq) * p.total_q + t] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
  }
}

}  // namespace

hipError_t launch_few_fwd(const bs_dims& dims, const void* q, const void* k, const void* v,
                          const int32_t* cu_q, const int32_t* cu_k, int32_t num_seqs,
                          int32_t max_seqlen, int causal, float scale, void* out, float* lse,
                          void* hdr, void* buf, const FewLayout& F, hipStream_t stream) {
  FewParams p;
  p.q = static_cast<const bf16*>(q);
  p.k = static_cast<const bf16*>(k);
  p.v = static_cast<const bf16*>(v);
  p.o = static_cast<bf16*>(out);
  p.lse = lse;
  p.cu_q = cu_q;
  p.cu_k = cu_k;
  p.hdr = static_cast<WsHeader*>(hdr);
  char* b = static_cast<char*>(buf);
  p.part = reinterpret_cast<float*>(b + F.part);
  p.stat = reinterpret_cast<float2*>(b + F.stat);
  p.cnt = F.slabs > 1 ? reinterpret_cast<int32_t*>(b) : nullptr;
  p.total_q = dims.total_q;
  p.total_k = dims.total_k;
  p.num_seqs = num_seqs;
  p.max_seqlen = max_seqlen;
  p.hq = dims.hq;
  p.hkv = dims.hkv;
  p.group = dims.hq / dims.hkv;
  p.causal = causal;
  p.slabs = F.slabs;
  p.per_min = F.per_min;
  p.scale_log2 = scale * kLog2e;
  const dim3 grid((unsigned)F.blocks), mgrid((unsigned)((dims.total_q * dims.hq * (dims.head_dim / 4) + 255) / 256));
  // keys read once (one row block per segment on average) go past the caches; where several row
  // blocks read them, the later ones find them there
  const bool once = dims.total_q * p.group <= 32 * (int64_t)num_seqs;
#define BS_FEW(D)                                                                              \
  do {                                                                                         \
    if (once) hipLaunchKernelGGL((few_fwd_kernel<D, 2>), grid, dim3(256), 0, stream, p);       \
    else hipLaunchKernelGGL((few_fwd_kernel<D, 0>), grid, dim3(256), 0, stream, p);            \
    if (F.slabs > 1) hipLaunchKernelGGL(few_merge_kernel<D>, mgrid, dim3(256), 0, stream, p);  \
  } while (0)
  if (dims.head_dim == 128) BS_FEW(128); else BS_FEW(64);
#undef BS_FEW
  return hipGetLastError();
}

}  // namespace bs
