// Softmax cross-entropy over a large vocabulary with its gradient fused in (Sec. 7,
// Fused SoftmaxCrossEntropy): bf16 (or fp32) logits in, fp32 arithmetic, per-token loss and
// log-sum-exp out, and the gradient g (softmax - onehot) written in the logits' dtype, in
// place over the logits if the caller wants.  No fp32 copy of the logits is ever made.
//
// Bandwidth-bound: each logit is read once and its gradient written once.  One workgroup per
// row; its lanes hold the row in registers, in 16-byte chunks, from the one read to the write
// of the gradient, and as a chunk's gradient is stored the same registers load that chunk of
// the workgroup's next row (the grid is persistent), so the next row's reads overlap this
// row's writes and arithmetic without extra registers.
//   - The lanes and chunks per lane follow the row: 256 lanes x 2 or 8 chunks, 512 x 8, 1024 x 8
//     or 16.  A short row on 1024 lanes leaves the memory idle while its sums are combined;
//     several small workgroups on a CU cover for one another.  Rows of 4,096 / 16,384 bf16
//     entries (8,192 rows) ran at 1.3 / 2.7 TB/s on one 1024-lane workgroup per CU.
//   - A row longer than 1024 x 16 chunks (131,072 bf16 entries) keeps that much in registers (3
//     chunks per lane where rows are few: the rule is at the launch) and reads the rest twice,
//     the second time from the caches.
//   - Rows of any length and alignment: the chunks start at the row's first 16-byte boundary,
//     and the up to 2 x (16 / size - 1) entries before and after them are held one per lane.
//     (One entry per lane and load, as odd vocabularies went before, ran at 1.9 TB/s at 2,048 x
//     32,003.)  Logits and gradient must lie alike modulo 16 bytes; where they do not, one entry
//     per lane is streamed twice (xent_stream_kernel).
// Measured, us before -> now (8,192 rows x 4,096: 104 -> 27; x 16,384: 197 -> 102; 2,048 x 32,003:
// 137 -> 55; x 50,257: 150 -> 85; x 152,064: 284 -> 261; float32 2,048 x 32,000: 129 -> 103; x
// 128,256: 499 -> 437; 4,096 x 128,256: 410 -> 404, 5.2 TB/s where a plain copy moves 4.9).
// Sums: every wave takes the maximum of its entries first, then sums 2^(x - max); lanes, then
// waves through LDS, are combined in a fixed order, so every run gives the same bits.
#include "common.hpp"

namespace bs {
namespace {

constexpr float kXentRescale = 8.0f;  // log2 units

struct XentParams {
  const void* logits;
  const int64_t* labels;
  void* dlogits;
  float* loss;
  float* lse;
  int64_t vocab;
  int64_t ignore_index;
  float grad_scale;
};

template <typename T> struct XVec;
template <> struct XVec<bf16> { typedef bf16x8 type; static constexpr int N = 8; };
template <> struct XVec<float> { typedef f32x4 type; static constexpr int N = 4; };

// Reductions over the 64 lanes in the vector unit (every lane gets the result): DPP inside rows
// of 16 lanes, then swaps of 16- and 32-lane halves.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <typename F>
__device__ __forceinline__ float row16_reduce(float x, F f) {
  x = f(x, dpp<0xB1>(x));   // lanes ^ 1
  x = f(x, dpp<0x4E>(x));   // lanes ^ 2
  x = f(x, dpp<0x141>(x));  // mirrored halves of 8
  x = f(x, dpp<0x140>(x));  // mirrored rows of 16
  return x;
}
template <typename F>
__device__ __forceinline__ float wave_reduce(float x, F f) {
  x = row16_reduce(x, f);
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float wave_max(float x) {
  return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float x) {
  return wave_reduce(x, [](float a, float b) { return a + b; });
}

// (max, sum) of the NW <= 16 waves of a workgroup, in log2 units; every lane of every wave gets
// log2 of the sum of 2^x.  red: 2 x 16 floats that nothing else uses until the next barrier but
// one.
template <int NW>
__device__ __forceinline__ float block_lse2(float m, float s, float (*red)[16], int lane, int w) {
  if (lane == 0) {
    red[0][w] = m;
    red[1][w] = s;
  }
  __syncthreads();
  const int i = lane & 15;
  const float mi = i < NW ? red[0][i] : -INFINITY;
  float si = i < NW ? red[1][i] : 0.f;
  const float M = row16_reduce(mi, [](float a, float b) { return fmaxf(a, b); });
  si *= mi == -INFINITY ? 1.f : fast_exp2(mi - M);  // an empty wave has sum 0 (or NaN)
  const float S = row16_reduce(si, [](float a, float b) { return a + b; });
  return M == -INFINITY ? -INFINITY : M + log2f(S);
}

// Adds N logits (raw values z; x = z log2 e) to the lane's running pair; the maximum is only
// raised when a chunk exceeds it by 2^8.
template <int N>
__device__ __forceinline__ void accumulate(const float (&z)[N], float& m, float& s) {
  float zc = z[0];
#pragma unroll
  for (int k = 1; k < N; ++k) zc = fmaxf(zc, z[k]);
  const float mc = zc * kLog2e;
  if (mc > m + kXentRescale) {  // first chunk (m = -inf), or a new max well above the old
    s *= fast_exp2(m - mc);
    m = mc;
  }
  const float b = m == -INFINITY ? 0.f : m;  // a row that so far holds only -inf
#pragma unroll
  for (int k = 0; k < N; ++k) s += fast_exp2(fmaf(z[k], kLog2e, -b));
}

template <typename T>
__device__ __forceinline__ void unpack(u32x4 x, float (&z)[XVec<T>::N]) {
  const typename XVec<T>::type v = __builtin_bit_cast(typename XVec<T>::type, x);
#pragma unroll
  for (int k = 0; k < XVec<T>::N; ++k) z[k] = (float)v[k];
}
template <typename T>
__device__ __forceinline__ T narrow(float x) {
  if constexpr (sizeof(T) == 2) return f2bf(x);
  else return x;
}

// f(chunk, index) for the chunks c, c + NT, ... below nb of a row, loaded in groups of U.
template <typename T, int NT, typename F>
__device__ __forceinline__ void stream_tail(const typename XVec<T>::type* src, int c, int nb, F f) {
  constexpr int U = 4;
  for (; c + (U - 1) * NT < nb; c += U * NT) {
    u32x4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = __builtin_bit_cast(u32x4, src[c + u * NT]);
#pragma unroll
    for (int u = 0; u < U; ++u) f(x[u], c + u * NT);
  }
  for (; c < nb; c += NT) f(__builtin_bit_cast(u32x4, src[c]), c);
}

// Waves per SIMD: at up to 8 chunks per lane (64 registers) the CU's 2,048 lanes are filled.
constexpr int xent_waves(int cpt) { return cpt <= 8 ? 8 : 4; }
constexpr int xent_blocks_per_cu(int nt, int waves) { return waves * 256 / nt; }

template <typename T, int NT, int CPT, bool kTail, int kWaves>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kWaves)))
void xent_kernel(const XentParams p, int64_t rows) {
  constexpr int N = XVec<T>::N, NW = NT / 64;
  typedef typename XVec<T>::type V;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* z0 = static_cast<const T*>(p.logits);
  T* d0 = static_cast<T*>(p.dlogits);
  __shared__ float red[2][2][16];  // alternating by row

  // a row's entries: `head` before the first 16-byte boundary, nb chunks, `extra` - head after
  struct Row {
    int64_t off;  // its first chunk, entries from the start of the logits
    int nb, head, extra;
  };
  auto row_of = [&](int64_t r) {
    Row g;
    const int mis = (int)((reinterpret_cast<uintptr_t>(z0 + r * p.vocab) & 15) / sizeof(T));
    g.head = (int)min((int64_t)((N - mis) & (N - 1)), p.vocab);
    g.nb = (int)(p.vocab - g.head) / N;
    g.extra = (int)p.vocab - g.nb * N;
    g.off = r * p.vocab + g.head;
    return g;
  };
  // position in the row of lane `tid`'s entry outside the chunks (tid < extra)
  auto extra_at = [&](const Row& g) {
    return tid < g.head ? tid : (int)p.vocab - g.extra + tid;
  };
  // buffer over the chunks held in registers: chunk i of the lane is at byte (tid + i NT) 16;
  // reads past the end give 0, writes are dropped
  auto rsrc_of = [&](const T* base, const Row& g) {
    const int n = min(g.nb, NT * CPT);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base + g.off), 0, (uint32_t)(n * 16), 0x00020000);
  };

  // some lane of this wave has a chunk i (a scalar test: rows need not fill the form)
  auto any = [&](int i, const Row& g) { return w * 64 + i * NT < g.nb; };

  int64_t row = blockIdx.x;
  u32x4 buf[CPT];
  float ex = 0.f;
  int64_t y = 0;
  Row g = {};
  if (row < rows) {
    g = row_of(row);
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(z0, g);
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      if (any(i, g)) buf[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, tid * 16, i * NT * 16, 0);
    if (tid < g.extra) ex = (float)z0[row * p.vocab + extra_at(g)];
    y = p.labels[row];
  }
  for (int it = 0; row < rows; ++it, row += gridDim.x) {
    const int64_t next = row + gridDim.x;
    const bool more = next < rows;
    const bool ignored = y == p.ignore_index;
    const bool in_range = y >= 0 && y < p.vocab;
    const bool labelled = in_range && !ignored;

    // the chunks beyond the registers first (their loads queue behind those of the registers):
    // the lane's running (max, sum); then the wave's maximum over everything, then the sum
    float ml = tid < g.extra ? ex * kLog2e : -INFINITY, s = 0.f;
    const V* tail = reinterpret_cast<const V*>(z0 + g.off);
    float tail_max = -INFINITY;
    if constexpr (kTail)
      stream_tail<T, NT>(tail, NT * CPT + tid, g.nb, [&](u32x4 x, int) {
        float z[N];
        unpack<T>(x, z);
        accumulate<N>(z, tail_max, s);
      });
    float mr = -INFINITY;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      if (any(i, g) && tid + i * NT < g.nb) {
        float z[N];
        unpack<T>(buf[i], z);
#pragma unroll
        for (int k = 0; k < N; ++k) mr = fmaxf(mr, z[k]);
      }
    }
    ml = fmaxf(ml, mr * kLog2e);
    if constexpr (kTail) ml = fmaxf(ml, tail_max);
    const float m = wave_max(ml);
    const float b = m == -INFINITY ? 0.f : m;
    if constexpr (kTail) s = tail_max == -INFINITY ? s : s * fast_exp2(tail_max - b);
    if (tid < g.extra) s += fast_exp2(fmaf(ex, kLog2e, -b));
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      // converted afresh here and below: fp32 copies would double the row's registers
      asm volatile("" : "+v"(buf[i]));
      if (any(i, g) && tid + i * NT < g.nb) {
        float z[N];
        unpack<T>(buf[i], z);
#pragma unroll
        for (int k = 0; k < N; ++k) s += fast_exp2(fmaf(z[k], kLog2e, -b));
      }
    }
    s = wave_sum(s);
    const float lse2 = block_lse2<NW>(m, s, red[it & 1], lane, w);
    if (tid == 0) {
      if (p.lse != nullptr) p.lse[row] = lse2 * kLn2;
      if (!labelled) p.loss[row] = ignored ? 0.f : NAN;
    }

    // gradient g (2^(x - lse2) - [j == label]) (zeros for an ignored row); the lane that holds
    // the label's logit writes the loss
    const bool grad = p.dlogits != nullptr;
    const float gs = p.grad_scale;
    const int at = labelled ? (int)y - g.head : -1;  // the label relative to the first chunk
    const bool in_chunks = at >= 0 && at < g.nb * N;
    const int cy = in_chunks ? at / N : -1, ky = at & (N - 1);
    auto grad_of = [&](float z) { return fast_exp2(fmaf(z, kLog2e, -lse2)) * gs; };
    auto chunk = [&](u32x4 x, int c) {
      float z[N];
      unpack<T>(x, z);
      float v[N];
#pragma unroll
      for (int k = 0; k < N; ++k) v[k] = grad_of(z[k]);
      if (c == cy) {
        float zy = z[0];
#pragma unroll
        for (int k = 1; k < N; ++k) zy = k == ky ? z[k] : zy;
        p.loss[row] = lse2 * kLn2 - zy;
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = k == ky ? v[k] - gs : v[k];
      }
      V o;
#pragma unroll
      for (int k = 0; k < N; ++k) o[k] = narrow<T>(v[k]);
      if (ignored) o = V{};  // uniform
      return __builtin_bit_cast(u32x4, o);
    };
    if (tid < g.extra) {
      const int e = extra_at(g);
      const bool is_label = labelled && e == (int)y;
      if (is_label) p.loss[row] = lse2 * kLn2 - ex;
      const float v = is_label ? grad_of(ex) - gs : grad_of(ex);
      if (grad) d0[row * p.vocab + e] = narrow<T>(ignored ? 0.f : v);
    }
    if constexpr (kTail) {
      if (grad) {
        V* dt = reinterpret_cast<V*>(d0 + g.off);
        stream_tail<T, NT>(tail, NT * CPT + tid, g.nb, [&](u32x4 x, int c) {
          dt[c] = __builtin_bit_cast(V, chunk(x, c));
        });
      } else if (cy >= NT * CPT && tid == 0) {
        p.loss[row] = lse2 * kLn2 - (float)z0[row * p.vocab + y];
      }
    }
    const Row gn = row_of(more ? next : row);
    const __amdgpu_buffer_rsrc_t ws = rsrc_of(grad ? d0 : const_cast<T*>(z0), g), rn = rsrc_of(z0, gn);
    if (more) {
      y = p.labels[next];
      if (tid < gn.extra) ex = (float)z0[next * p.vocab + extra_at(gn)];
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      asm volatile("" : "+v"(buf[i]));
      if (any(i, g) && (grad || tid + i * NT == cy)) {
        const u32x4 o = chunk(buf[i], tid + i * NT);
        if (grad) __builtin_amdgcn_raw_buffer_store_b128(o, ws, tid * 16, i * NT * 16, 0);
      }
      // the same registers take this chunk of the next row (its read overlaps these writes)
      if (more && any(i, gn)) buf[i] = __builtin_amdgcn_raw_buffer_load_b128(rn, tid * 16, i * NT * 16, 0);
    }
    g = gn;
  }
}

// Logits and gradient that lie differently modulo 16 bytes: one entry per lane and step, the
// row streamed twice by a persistent grid (one workgroup per CU) that finds it in the caches
// the second time.
constexpr int kStreamThreads = 1024;
template <typename T>
__global__ __launch_bounds__(kStreamThreads) void xent_stream_kernel(const XentParams p, int64_t rows) {
  constexpr int U = 8, NT = kStreamThreads;  // entries in flight per lane
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  __shared__ float red[2][2][16];
  int it = 0;
  for (int64_t row = blockIdx.x; row < rows; row += gridDim.x, ++it) {
    const T* zr = static_cast<const T*>(p.logits) + row * p.vocab;
    const int64_t y = p.labels[row];
    const bool ignored = y == p.ignore_index;
    const bool in_range = y >= 0 && y < p.vocab;
    float ml = -INFINITY, s = 0.f;
    int64_t c = tid;
    for (; c + (U - 1) * NT < p.vocab; c += U * NT) {
      float z[U];
#pragma unroll
      for (int u = 0; u < U; ++u) z[u] = (float)zr[c + u * NT];
      accumulate<U>(z, ml, s);
    }
    for (; c < p.vocab; c += NT) {
      const float z[1] = {(float)zr[c]};
      accumulate<1>(z, ml, s);
    }
    const float m = wave_max(ml);
    s = wave_sum(ml == -INFINITY ? s : s * fast_exp2(ml - m));
    const float lse2 = block_lse2<NT / 64>(m, s, red[it & 1], lane, w);
    if (tid == 0) {
      if (p.lse != nullptr) p.lse[row] = lse2 * kLn2;
      p.loss[row] = ignored ? 0.f : (in_range ? lse2 * kLn2 - (float)zr[y] : NAN);
    }
    T* dr = static_cast<T*>(p.dlogits) + row * p.vocab;
    const float g = p.grad_scale;
    if (ignored) {
      for (c = tid; c < p.vocab; c += NT) dr[c] = narrow<T>(0.f);
      continue;
    }
    auto grad = [&](float z, int64_t at) {
      const float v = fast_exp2(fmaf(z, kLog2e, -lse2)) * g;
      dr[at] = narrow<T>(at == y ? v - g : v);
    };
    // U loads in flight here too (one at a time / so: 100 x 200,003 bf16 89 / 38 us, 1,000 x 50,257
    // 89 / 50; float32 92 / 46 and 125 / 101)
    for (c = tid; c + (U - 1) * NT < p.vocab; c += U * NT) {
      float z[U];
#pragma unroll
      for (int u = 0; u < U; ++u) z[u] = (float)zr[c + u * NT];
#pragma unroll
      for (int u = 0; u < U; ++u) grad(z[u], c + u * NT);
    }
    for (; c < p.vocab; c += NT) grad((float)zr[c], c);
  }
}

template <typename T>
hipError_t launch_xent(const XentParams& p, int64_t rows, hipStream_t stream) {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess)
    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  auto blocks = [&](int64_t per_cu) {
    return dim3((unsigned)(rows < cus * per_cu ? rows : cus * per_cu));
  };
  const bool alike = p.dlogits == nullptr || ((reinterpret_cast<uintptr_t>(p.logits) ^
                                               reinterpret_cast<uintptr_t>(p.dlogits)) & 15) == 0;
  if (!alike) {
    hipLaunchKernelGGL(xent_stream_kernel<T>, blocks(1), dim3(kStreamThreads), 0, stream, p, rows);
    return hipGetLastError();
  }
#define BS_XENT_W(NT, CPT, TAIL, WAVES)                                                         \
  hipLaunchKernelGGL((xent_kernel<T, NT, CPT, TAIL, WAVES>), blocks(xent_blocks_per_cu(NT, WAVES)), \
                     dim3(NT), 0, stream, p, rows)
#define BS_XENT(NT, CPT, TAIL) BS_XENT_W(NT, CPT, TAIL, xent_waves(CPT))
  const int64_t nch = p.vocab / XVec<T>::N;  // chunks of a row at most
  // a long bf16 row for at most every other CU: no row overlaps another, and what counts is one
  // workgroup's work per entry, which streaming needs less of (64 x 200,000 with / without the
  // gradient: 27.3 / 13.8 us by the forms below, 24.9 / 13.0 so; 200 x 152,064: 26.9 / 13.4 below)
  if constexpr (sizeof(T) == 2)
    if (nch > 16384 && rows * 2 <= cus) {
      BS_XENT_W(1024, 3, true, 4);
      return hipGetLastError();
    }
  if (nch <= 512) BS_XENT(256, 2, false);
  else if (nch <= 2048) BS_XENT(256, 8, false);
  else if (nch <= 4096) BS_XENT(512, 8, false);
  else if (nch <= 8192) BS_XENT(1024, 8, false);
  // the loss alone reads each entry once anyway: two workgroups per CU instead of registers
  // (2,048 x 200,000: 138 us against 143 with one)
  else if (p.dlogits == nullptr) BS_XENT(1024, 2, true);
  else if (nch <= 16384) BS_XENT(1024, 16, false);
  else BS_XENT(1024, 16, true);
#undef BS_XENT
#undef BS_XENT_W
  return hipGetLastError();
}

}  // namespace

hipError_t launch_softmax_xent(int64_t rows, int64_t vocab, int dtype, const void* logits,
                               const int64_t* labels, int64_t ignore_index, float grad_scale,
                               float* loss, float* lse, void* dlogits, hipStream_t stream) {
  if (rows == 0) return hipSuccess;
  XentParams p;
  p.logits = logits;
  p.labels = labels;
  p.dlogits = dlogits;
  p.loss = loss;
  p.lse = lse;
  p.vocab = vocab;
  p.ignore_index = ignore_index;
  p.grad_scale = grad_scale;
  return dtype == BS_BF16 ? launch_xent<bf16>(p, rows, stream) : launch_xent<float>(p, rows, stream);
}

}  // namespace bs
