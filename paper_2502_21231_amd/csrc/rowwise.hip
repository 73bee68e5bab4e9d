// Bandwidth-bound row kernels: LSE merge, dQ finalize, and the sums over the parts of a split
// chain (few_bf16.hip has its own, over a varying number of pieces).
//
// Each (token, head) row of head_dim elements is handled by a group of
// head_dim/8 (bf16) or head_dim/4 (fp32) lanes, one 16-byte vector per lane,
// so every row is read and written with fully coalesced 16-byte accesses.
#include "attn.hpp"

namespace bs {
namespace {

template <typename T> struct Vec;
template <> struct Vec<bf16> { typedef bf16x8 type; static constexpr int N = 8; };
template <> struct Vec<float> { typedef f32x4 type; static constexpr int N = 4; };

template <typename T>
__device__ __forceinline__ float to_f(T x) { return (float)x; }
template <typename T>
__device__ __forceinline__ T from_f(float x);
template <> __device__ __forceinline__ bf16 from_f<bf16>(float x) { return f2bf(x); }
template <> __device__ __forceinline__ float from_f<float>(float x) { return x; }

// Combination of the partial results of one query row over n disjoint key
// sets (the steps of a context-parallel ring):
//   LSE = m + log(sum_c exp(LSE_c - m)),   O = sum_c exp(LSE_c - LSE) O_c,
// m = max_c LSE_c; partials at -inf weigh 0; all -inf gives O = 0, LSE = -inf.
template <typename T, int D, int U, bool kByXcd>
__global__ __launch_bounds__(256) void lse_merge_kernel(const T* __restrict__ parts,
                                                        const float* __restrict__ lse_parts,
                                                        int32_t n, int64_t rows, int32_t hq,
                                                        int64_t total_q, T* __restrict__ out,
                                                        float* __restrict__ lse) {
  typedef typename Vec<T>::type V;
  constexpr int LPR = D / Vec<T>::N;  // lanes per row
  // Blocks are dealt to the 8 XCDs round-robin; with kByXcd each XCD takes a contiguous eighth of
  // the rows, so that a line of the LSE (one head, 32 tokens) comes into one XCD's L2, not into
  // eight (bf16, n = 8, 8,192 tokens, 32 heads: 108.2 -> 103.4 us, 5.9 TB/s; n = 2, 48 heads: 55.7 ->
  // 49.8).  The rule and where it does not pay are at the launch.
  const int64_t blk = kByXcd ? (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  const int64_t gid = blk * blockDim.x + threadIdx.x;
  const int64_t row = gid / LPR;      // row = t * hq + h
  const int part = gid % LPR;
  if (row >= rows) return;
  const int64_t t = row / hq;
  const int h = row % hq;
  const float* lp = lse_parts + (int64_t)h * total_q + t;
  const int64_t lstride = (int64_t)hq * total_q;
  const int64_t pstride = rows * D;
  const T* src = parts + row * D + part * Vec<T>::N;
  float acc[Vec<T>::N];
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) acc[i] = 0.f;
  float m = -INFINITY, wsum = 0.f;
  // partials in groups of U: every load of a group is issued before any of it is used, so
  // that each lane keeps U row reads in flight (one at a time is latency-bound); the sum is
  // rescaled when a group raises the running maximum
  for (int c0 = 0; c0 < n; c0 += U) {
    float l[U];
    V x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + u < n) {
        l[u] = lp[(c0 + u) * lstride];
        x[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(src + (c0 + u) * pstride));
      } else {
        l[u] = -INFINITY;
        x[u] = V{};
      }
    }
    float mg = m;
#pragma unroll
    for (int u = 0; u < U; ++u) mg = fmaxf(mg, l[u]);
    if (mg == -INFINITY) continue;
    const float r = expf(m - mg);  // 0 while nothing was added (m = -inf)
    wsum *= r;
#pragma unroll
    for (int i = 0; i < Vec<T>::N; ++i) acc[i] *= r;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float wgt = expf(l[u] - mg);  // exp(-inf) = 0
      wsum += wgt;
#pragma unroll
      for (int i = 0; i < Vec<T>::N; ++i) acc[i] += wgt * to_f(x[u][i]);
    }
    m = mg;
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  V y;
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) y[i] = from_f<T>(acc[i] * inv);
  __builtin_nontemporal_store(y, reinterpret_cast<V*>(out + row * D + part * Vec<T>::N));
  if (part == 0) lse[(int64_t)h * total_q + t] = m == -INFINITY ? -INFINITY : m + logf(wsum);
}

template <typename T>
__global__ __launch_bounds__(256) void dq_finalize_kernel(const float* __restrict__ acc,
                                                          T* __restrict__ dq, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const f32x4 x = reinterpret_cast<const f32x4*>(acc)[i];
  T y[4] __attribute__((aligned(16)));
#pragma unroll
  for (int j = 0; j < 4; ++j) y[j] = from_f<T>(x[j]);
  if constexpr (sizeof(T) == 2)
    *reinterpret_cast<bf16x4*>(dq + i * 4) = *reinterpret_cast<const bf16x4*>(y);
  else
    *reinterpret_cast<f32x4*>(dq + i * 4) = *reinterpret_cast<const f32x4*>(y);
}

// Forward of split chains: O = sum_s 2^(M_s - M) O_s / L, LSE = (M + log2 L) ln 2 with
// L = sum_s 2^(M_s - M) L_s, written as bf16 or folded into the running state as the forward's
// epilogue does.  head_dim / 4 lanes per (token, head) row; at most 8 parts, all loads first.
constexpr int kMaxSplits = 8;
template <int D>
__global__ __launch_bounds__(256) void fwd_combine_kernel(const float* __restrict__ part, int splits,
                                                          int64_t total_q, int32_t hq, bf16* out,
                                                          float* lse, float* o_run, float* lse_run,
                                                          int accumulate, const WsHeader* hdr) {
  if (hdr->status != BS_DEV_OK) return;  // the segments were rejected
  constexpr int LPR = D / 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t rows = total_q * hq, row = gid / LPR;
  const int ch = (int)(gid % LPR);
  if (row >= rows) return;
  const float2* stat = reinterpret_cast<const float2*>(part + splits * rows * D);
  float m[kMaxSplits], l[kMaxSplits];
  f32x4 x[kMaxSplits];
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int i = 0; i < kMaxSplits; ++i) {
    m[i] = -INFINITY;
    l[i] = 0.f;
    x[i] = f32x4{};
    if (i < splits) {
      const float2 st = stat[i * rows + row];
      m[i] = st.x;
      l[i] = st.y;
      x[i] = *reinterpret_cast<const f32x4*>(part + (i * rows + row) * D + ch * 4);
    }
    M = fmaxf(M, m[i]);
  }
  const float base = M == -INFINITY ? 0.f : M;
  f32x4 o = f32x4{};
#pragma unroll
  for (int i = 0; i < kMaxSplits; ++i) {
    const float w = fast_exp2(m[i] - base);
    L += l[i] * w;
    if (i < splits) o += x[i] * w;
  }
  o *= L > 0.f ? 1.f / L : 0.f;
  const float lse2 = L > 0.f ? M + log2f(L) : -INFINITY;  // log2 units
  const int64_t t = row / hq, li = (row - t * hq) * total_q + t;
  bf16x4* ob = reinterpret_cast<bf16x4*>(out + row * D + ch * 4);
  if (o_run == nullptr) {
    *ob = bf16x4{f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3])};
    if (ch == 0) lse[li] = lse2 * kLn2;
    return;
  }
  const float old2 = accumulate ? lse_run[li] * kLog2e : -INFINITY;
  const float mx = fmaxf(old2, lse2);
  float w_old = 0.f, w_new = 0.f, lse_m = -INFINITY;
  if (mx != -INFINITY) {
    const float eo = fast_exp2(old2 - mx), en = fast_exp2(lse2 - mx);
    w_old = eo / (eo + en);
    w_new = en / (eo + en);
    lse_m = (mx + log2f(eo + en)) * kLn2;
  }
  o *= w_new;
  f32x4* orun = reinterpret_cast<f32x4*>(o_run + row * D + ch * 4);
  if (w_old != 0.f) o += *orun * w_old;
  if (out != nullptr) *ob = bf16x4{f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3])};
  else *orun = o;
  __builtin_amdgcn_wave_barrier();  // every lane of the row has read the old LSE
  if (ch == 0) lse_run[li] = lse_m;
}

// out (z = 0: out0, 1: out1) = sum over the slabs, four floats per lane.
__global__ __launch_bounds__(256) void sum_slabs_kernel(const float* __restrict__ part, int splits,
                                                        int64_t n4, void* out0, void* out1,
                                                        int mode, const WsHeader* hdr) {
  if (hdr->status != BS_DEV_OK) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const f32x4* src = reinterpret_cast<const f32x4*>(part) + (int64_t)blockIdx.y * splits * n4 + i;
  f32x4 x[kMaxSplits];
#pragma unroll
  for (int s = 0; s < kMaxSplits; ++s)
    if (s < splits) x[s] = src[s * n4];
  f32x4 y = x[0];
#pragma unroll
  for (int s = 1; s < kMaxSplits; ++s)
    if (s < splits) y += x[s];
  void* out = blockIdx.y == 0 ? out0 : out1;
  if (mode != kSumBf16) {
    f32x4* dst = static_cast<f32x4*>(out) + i;
    *dst = mode == kSumAddF32 ? *dst + y : y;
  } else {
    static_cast<bf16x4*>(out)[i] = bf16x4{f2bf(y[0]), f2bf(y[1]), f2bf(y[2]), f2bf(y[3])};
  }
}

inline unsigned blocks_for(int64_t threads) { return (unsigned)((threads + 255) / 256); }

}  // namespace

hipError_t launch_lse_merge(const bs_dims& dims, const void* out_parts, const float* lse_parts,
                            int32_t n, void* out, float* lse, hipStream_t stream) {
  const int64_t rows = dims.total_q * dims.hq;
  if (rows == 0) return hipSuccess;
  const int vec = dims.dtype == BS_BF16 ? 8 : 4;
  const unsigned grid = (blocks_for(rows * (dims.head_dim / vec)) + 7) / 8 * 8;
  // rows of 512 bytes, 64K of them or more: the lines of the LSE are then little of the traffic, and
  // eight streams far apart cost more (float32, head_dim 128, round / by XCD: n = 2, 8,192 tokens, 32
  // heads 62.4 / 65.8 us; n = 8, 4,096 tokens 98.3 / 101.4; n = 16, 1,024 tokens, 16 heads 23.4 / 22.2;
  // head_dim 64, n = 4, 16,384 tokens, 8 heads 28.7 / 27.0)
  const bool by_xcd = rows < 65536;
#define BS_MERGE_U(T, D, U, X)                                                                \
  hipLaunchKernelGGL((lse_merge_kernel<T, D, U, X>), dim3(grid), dim3(256), 0, stream,       \
                     static_cast<const T*>(out_parts), lse_parts, n, rows, dims.hq,           \
                     dims.total_q, static_cast<T*>(out), lse)
#define BS_MERGE(T, D, X)                                                                     \
  do {                                                                                        \
    if (n <= 2) BS_MERGE_U(T, D, 2, X);                                                       \
    else if (n <= 4) BS_MERGE_U(T, D, 4, X);                                                  \
    else BS_MERGE_U(T, D, 8, X);                                                              \
  } while (0)
  if (dims.dtype == BS_BF16) {
    if (dims.head_dim == 128) BS_MERGE(bf16, 128, true); else BS_MERGE(bf16, 64, true);
  } else if (dims.head_dim == 64) {
    BS_MERGE(float, 64, true);
  } else {
    if (by_xcd) BS_MERGE(float, 128, true); else BS_MERGE(float, 128, false);
  }
#undef BS_MERGE
#undef BS_MERGE_U
  return hipGetLastError();
}

hipError_t launch_dq_finalize(const bs_dims& dims, const float* dq_acc, void* dq,
                              hipStream_t stream) {
  const int64_t n4 = dims.total_q * dims.hq * dims.head_dim / 4;
  if (n4 == 0) return hipSuccess;
  if (dims.dtype == BS_BF16)
    hipLaunchKernelGGL(dq_finalize_kernel<bf16>, dim3(blocks_for(n4)), dim3(256), 0, stream,
                       dq_acc, static_cast<bf16*>(dq), n4);
  else
    hipLaunchKernelGGL(dq_finalize_kernel<float>, dim3(blocks_for(n4)), dim3(256), 0, stream,
                       dq_acc, static_cast<float*>(dq), n4);
  return hipGetLastError();
}

hipError_t launch_fwd_combine(const bs_dims& dims, const SelfPlan& self, void* out, float* lse,
                              const FwdMerge* merge, hipStream_t stream) {
  const unsigned grid = blocks_for(dims.total_q * dims.hq * (dims.head_dim / 4));
#define BS_COMBINE(D)                                                                           \
  hipLaunchKernelGGL(fwd_combine_kernel<D>, dim3(grid), dim3(256), 0, stream, self.part,        \
                     self.splits, dims.total_q, dims.hq, static_cast<bf16*>(out), lse,          \
                     merge ? merge->o_run : nullptr, merge ? merge->lse_run : nullptr,          \
                     merge ? merge->accumulate : 0, self.plan.hdr)
  if (dims.head_dim == 128) BS_COMBINE(128); else BS_COMBINE(64);
#undef BS_COMBINE
  return hipGetLastError();
}

hipError_t launch_sum_slabs(const float* part, int splits, int64_t n, void* out0, void* out1,
                            SumOut mode, const WsHeader* hdr, hipStream_t stream) {
  hipLaunchKernelGGL(sum_slabs_kernel, dim3(blocks_for(n / 4), out1 != nullptr ? 2 : 1), dim3(256), 0,
                     stream, part, splits, n / 4, out0, out1, (int)mode, hdr);
  return hipGetLastError();
}

}  // namespace bs
