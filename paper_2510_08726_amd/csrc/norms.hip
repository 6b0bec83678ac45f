// Row reductions fused by rolling update and split by split-k update: the
// stable L2 norm and RMSNorm with the row max of its output (the paper's
// second workload; see include/norms.h).  Both are HBM streams: every lane
// reads 16-byte vectors of its row chunk in batches, folds each batch into
// its state with one repaired update (the batch's own max and sum first, the
// privatised local reduction), the lanes' states are combined with the same
// repair, and the chunk partials of a row are combined by a second kernel.
// With one chunk per row there is no second kernel: a row kernel (a wave or a
// workgroup per row, by the row's length) writes the norm, or, when the row
// fits in registers, y from them without reading X again.
//
// Ends of rows and chunks: a lane past the end loads the last vector again
// (no branches between the loads of a batch, which keeps all of them in
// flight) and leaves it out of its sums.
//
// Cache policy: X is read once by the L2 norm and by the one-pass RMSNorm,
// and last by RMSNorm's second kernel, so those loads are nontemporal, and
// so are the second kernel's stores of y; RMSNorm's first pass reads X with
// ordinary loads so that the second pass finds what the caches (L2 and the
// memory-side cache) still hold of it.  (The one-pass kernel's stores of y
// are ordinary: 1.5 % faster there.)

#include <type_traits>

#include "kernel_common.h"
#include "launch.h"

namespace attn {

namespace {

constexpr int kNormThreads = 256;
constexpr int kL2RowThreads = 256;   // the L2 norm with one chunk per row
constexpr int kL2RowUnroll = 16;     // its 16-byte loads in flight per lane
constexpr int kWaveRowVecs = 512;    // longest row (vectors) of the row kernels that one wave takes
constexpr int kRowThreads = 1024;    // the one-pass RMSNorm: most lanes of one row
constexpr int kRowVecs = (int)(kNormRowBytes / (kRowThreads * 16));   // most 16-byte vectors per lane
constexpr int kRowBatch = 2;         // of which 1024 lanes load (and fold) at a time
constexpr int kShareBatch = 4;       // and fewer lanes, whose workgroups share a compute unit
constexpr int kRowsToShare = 256;    // rows from which they do: one for each of the MI355X's 256 compute units
static_assert(kRowVecs % kRowBatch == 0 && kRowVecs % kShareBatch == 0, "whole batches");
constexpr int kNormUnroll = 8;    // 16-byte loads in flight per lane, first pass
constexpr int kFold = 4;          // vectors a lane folds in one update
constexpr int kApplyUnroll = 4;   // the same in RMSNorm's second pass

template <bool NT>
static __device__ __forceinline__ u32x4 load16(const u32x4* a) {
  if constexpr (NT) return __builtin_nontemporal_load(a);
  else return *a;
}

template <typename T> struct Vec;
template <> struct Vec<_Float16> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void load(const u32x4& w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t u = w[i];   // (a bit_cast of the element itself reads element 0 on this compiler)
      const f16x2 h = __builtin_bit_cast(f16x2, u);
      f[2 * i] = (float)h[0];
      f[2 * i + 1] = (float)h[1];
    }
  }
  static __device__ __forceinline__ u32x4 store(const float* f) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = Elem<_Float16>::pack2(f[2 * i], f[2 * i + 1]);
    return w;
  }
};
template <> struct Vec<__bf16> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void load(const u32x4& w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = Elem<__bf16>::lo(w[i]);
      f[2 * i + 1] = Elem<__bf16>::hi(w[i]);
    }
  }
  static __device__ __forceinline__ u32x4 store(const float* f) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = Elem<__bf16>::pack2(f[2 * i], f[2 * i + 1]);
    return w;
  }
};
template <> struct Vec<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void load(const u32x4& w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t u = w[i];   // as above
      f[i] = __builtin_bit_cast(float, u);
    }
  }
  static __device__ __forceinline__ u32x4 store(const float* f) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = f[i];
      w[i] = __builtin_bit_cast(uint32_t, x);
    }
    return w;
  }
};

// Sum and maximum over the 64 lanes of a wave, in every lane.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <typename F>
__device__ __forceinline__ float wave_reduce(float x, F&& f) {
  x = f(x, dpp_move<0xB1>(x));    // quad_perm [1,0,3,2]
  x = f(x, dpp_move<0x4E>(x));    // quad_perm [2,3,0,1]
  x = f(x, dpp_move<0x141>(x));   // row_half_mirror
  x = f(x, dpp_move<0x140>(x));   // row_mirror
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // rows 0, 1 and 2, 3
  const unsigned a0 = a[0], a1 = a[1];
  x = f(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1));
  const unsigned v = __builtin_bit_cast(unsigned, x);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // halves
  const unsigned b0 = b[0], b1 = b[1];
  return f(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}
__device__ __forceinline__ float wave_sum(float x) {
  return wave_reduce(x, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float x) {
  return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); });
}

// The rolling state of one lane and its two updates: fold K vectors of
// Vec<T>::N values (privatised: the batch's own reduction, then one repaired
// global update; vectors u with !ok(u) are repeats and not summed), and merge
// another state (the split-k combine of two partials).
//
// L2: r = max |x| so far, t = sum of (x / r)^2 so far.
struct L2State {
  float r = 0.f, t = 0.f;
  template <typename T, int K, typename OK>
  __device__ __forceinline__ void fold(const u32x4* w, OK&& ok, float, float) {
    // kFold vectors an update: enough to spread its division, few enough that
    // their converted values fit in registers between the two passes.
    constexpr int G = K < kFold ? K : kFold, VN = Vec<T>::N;
    static_assert(K % G == 0, "whole updates");
#pragma unroll
    for (int u0 = 0; u0 < K; u0 += G) {
      float c[G][VN], vm = 0.f;
#pragma unroll
      for (int u = 0; u < G; ++u) {
        Vec<T>::load(w[u0 + u], c[u]);
#pragma unroll
        for (int k = 0; k < VN; ++k) vm = fmaxf(vm, fabsf(c[u][k]));
      }
      const float rn = fmaxf(r, vm);
      const float inv = rn > 0.f ? 1.f / rn : 0.f;       // all zero so far: nothing to add
      const float a = r * inv;                           // h: t (r / r')^2
      t *= a * a;
#pragma unroll
      for (int u = 0; u < G; ++u) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < VN; ++k) {
          const float q = c[u][k] * inv;                 // g(r', c) = (c / r')^2
          s = __builtin_fmaf(q, q, s);
        }
        t += ok(u0 + u) ? s : 0.f;
      }
      r = rn;
    }
  }
  __device__ __forceinline__ void merge(float r2, float t2, float) {
    const float rn = fmaxf(r, r2);
    if (rn > 0.f) {
      const float a = r / rn, b = r2 / rn;
      t = t * a * a + t2 * b * b;
      r = rn;
    }
  }
  // Merge the states of a wave's 64 lanes, in every lane: the producer first,
  // then every consumer repaired to it at once (one division instead of two
  // in each of six steps).
  __device__ __forceinline__ void wave_merge(float) {
    const float rn = wave_max(r);
    const float a = rn > 0.f ? r / rn : 0.f;
    t = wave_sum(t * a * a);
    r = rn;
  }
};

// RMSNorm statistics: r = sum of x^2 / M so far (the running mean), t = max
// of x / sqrt(r + eps) so far.
struct RmsState {
  float r = 0.f, t = kNegInf;
  template <typename T, int K, typename OK>
  __device__ __forceinline__ void fold(const u32x4* w, OK&& ok, float invM, float eps) {
    constexpr int G = K < kFold ? K : kFold;
    static_assert(K % G == 0, "whole updates");
#pragma unroll
    for (int u0 = 0; u0 < K; u0 += G) {
      float rn = r, vm = kNegInf;
      sums<T, G>(w + u0, [&](int u) { return ok(u0 + u); }, invM, rn, vm);
      const float q = __builtin_amdgcn_rsqf(rn + eps);   // 1 / sqrt(r' + eps)
      // h(t, r, r') = t sqrt(r + eps) / sqrt(r' + eps); g(r', c) = c / sqrt(r' + eps).
      // Before the first value t is -inf and stays so under h (also when
      // r + eps = 0, where the factor would be 0).
      t = fmaxf(repair(t, r, q, eps), vm * q);
      r = rn;
    }
  }
  // The producer's sum and the plain maximum of K vectors.
  template <typename T, int K, typename OK>
  static __device__ __forceinline__ void sums(const u32x4* w, OK&& ok, float invM, float& r, float& vm) {
    constexpr int VN = Vec<T>::N;
#pragma unroll
    for (int u = 0; u < K; ++u) {
      float c[VN], s = 0.f, m = vm;
      Vec<T>::load(w[u], c);
#pragma unroll
      for (int k = 0; k < VN; ++k) {
        s = __builtin_fmaf(c[k], c[k], s);
        m = fmaxf(m, c[k]);
      }
      // A repeat counts in neither: its maximum without its squares would be
      // scaled by 1 / sqrt(eps), which can overflow.
      const bool in = ok(u);
      r = in ? __builtin_fmaf(s, invM, r) : r;
      vm = in ? m : vm;
    }
  }
  __device__ __forceinline__ void merge(float r2, float t2, float eps) {
    const float rn = r + r2;
    const float q = __builtin_amdgcn_rsqf(rn + eps);
    t = fmaxf(repair(t, r, q, eps), repair(t2, r2, q, eps));
    r = rn;
  }
  __device__ __forceinline__ void wave_merge(float eps) {
    const float rn = wave_sum(r);
    t = wave_max(repair(t, r, __builtin_amdgcn_rsqf(rn + eps), eps));
    r = rn;
  }
  // h(t, r, r') with q = 1 / sqrt(r' + eps).
  static __device__ __forceinline__ float repair(float t, float r, float q, float eps) {
    return t == kNegInf ? kNegInf : t * (__builtin_sqrtf(r + eps) * q);
  }
};

template <typename T, bool NT, int NTH, int UNR, typename S>
__device__ __forceinline__ void fold_chunk(const NormParams& p, int n, int c, S& st) {
  constexpr int VN = Vec<T>::N;
  // This chunk's vectors.
  const int v0 = (int)(min((long long)c * p.chunk, (long long)p.M) / VN);
  const int v1 = (int)(min((long long)(c + 1) * p.chunk, (long long)p.M) / VN);
  const u32x4* row = reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(p.x) + (size_t)n * p.M);
  const int tid = threadIdx.x;
  auto load = [&](auto& w, int b) {
    constexpr int K = sizeof(w) / sizeof(w[0]);
#pragma unroll
    for (int u = 0; u < K; ++u) w[u] = load16<NT>(row + min(b + tid + u * NTH, v1 - 1));
  };
  auto fold = [&](auto& w, int b) {
    constexpr int K = sizeof(w) / sizeof(w[0]);
    st.template fold<T, K>(w, [&](int u) { return b + tid + u * NTH < v1; }, p.invM, p.eps);
  };
  // Batches of UNR / 2 vectors a lane, the next one's loads issued before a
  // batch is folded; a chunk of at most two vectors a lane is one batch.  (The
  // last batch is a whole one too: read one load at a time it cost a memory
  // latency per vector.)
  constexpr int H = UNR / 2;
  if (v1 - v0 <= 2 * NTH) {
    if (v1 <= v0) return;
    u32x4 w[2];
    load(w, v0);
    fold(w, v0);
    return;
  }
  u32x4 wa[H], wb[H];
  load(wa, v0);
  for (int b = v0;;) {
    if (b + H * NTH < v1) load(wb, b + H * NTH);
    fold(wa, b);
    if ((b += H * NTH) >= v1) break;
    if (b + H * NTH < v1) load(wa, b + H * NTH);
    fold(wb, b);
    if ((b += H * NTH) >= v1) break;
  }
}

// Combine the states of the workgroup's NTH lanes (the same repaired merge),
// leaving the result in the lanes of wave 0.
template <int NTH, typename S>
__device__ __forceinline__ void block_merge(S& st, float eps) {
  __shared__ float sr[NTH / 64], stt[NTH / 64];
  st.wave_merge(eps);
  if ((threadIdx.x & 63) == 0) {
    sr[threadIdx.x >> 6] = st.r;
    stt[threadIdx.x >> 6] = st.t;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    st = S();
    if (threadIdx.x < NTH / 64) {
      st.r = sr[threadIdx.x];
      st.t = stt[threadIdx.x];
    }
    st.wave_merge(eps);
  }
}

// Local nests: one workgroup per (chunk c, row n) writes its partial (r, t).
template <typename T, bool RMS>
__global__ __launch_bounds__(kNormThreads) void norm_split_kernel(NormParams p) {
  const int c = blockIdx.x % p.chunks, n = blockIdx.x / p.chunks;
  typename std::conditional<RMS, RmsState, L2State>::type st;
  fold_chunk<T, !RMS, kNormThreads, kNormUnroll>(p, n, c, st);
  block_merge<kNormThreads>(st, p.eps);
  if (threadIdx.x == 0) {
    p.ws_r[blockIdx.x] = st.r;
    p.ws_t[blockIdx.x] = st.t;
  }
}

// One chunk per row, short rows: a wave holds RW whole rows of at most 64 V
// vectors, V a lane, with all loads in flight at once.
template <typename T, int V, int RW>
__device__ __forceinline__ void load_rows(const NormParams& p, int n0, int nv, u32x4 (&w)[RW][V]) {
  const u32x4* x = reinterpret_cast<const u32x4*>(p.x);
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < RW; ++i)
#pragma unroll
    for (int u = 0; u < V; ++u)
      w[i][u] = load16<true>(x + (size_t)min(n0 + i, p.N - 1) * nv + min(lane + 64 * u, nv - 1));
}

template <typename T, int V, int RW>
__device__ __forceinline__ void l2_wave_rows(const NormParams& p, int nv) {
  const int lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * (kL2RowThreads / 64) + (threadIdx.x >> 6)) * RW;
  if (n0 >= p.N) return;
  u32x4 w[RW][V];
  load_rows<T, V, RW>(p, n0, nv, w);
  float r[RW], t[RW];
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    L2State st;
    st.fold<T, V>(w[i], [&](int u) { return lane + 64 * u < nv; }, 0.f, 0.f);
    st.wave_merge(0.f);
    r[i] = st.r;
    t[i] = st.t;
  }
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < RW; ++i)
      if (n0 + i < p.N) {
        p.ws_r[n0 + i] = r[i];
        p.ws_t[n0 + i] = t[i];
        p.out[n0 + i] = r[i] * __builtin_sqrtf(t[i]);
      }
  }
}

// The L2 norm with one chunk per row: a wave per row up to kWaveRowVecs
// vectors (8192 x 1024 bf16: 4.7 us, 14.4 with a workgroup a row), else one
// workgroup of 256 lanes per row with two batches of 8 loads a lane, one in
// flight while the other is folded (256 x 2^17 fp32 rows: 21.9 us, 6.13 TB/s,
// against 24.5 with 512 lanes, 32 with 1024, and 23.3 with 16 loads folded
// before the next 16; 500 x 30000 bf16: 6.9 us, 12.9 with the row's tail read
// one load at a time); it writes the row's partial and its norm.  At most 128
// registers, so that 16 waves share a compute unit.
template <typename T>
__global__ __launch_bounds__(kL2RowThreads, 4) void l2_row_kernel(NormParams p) {
  const int nv = p.M / Vec<T>::N;
  if (p.lanes == 64) {
    if (nv <= 64) l2_wave_rows<T, 1, 1>(p, nv);
    else if (nv <= 128) l2_wave_rows<T, 2, 1>(p, nv);
    else if (nv <= 256) l2_wave_rows<T, 4, 1>(p, nv);
    else l2_wave_rows<T, 8, 1>(p, nv);
    return;
  }
  const int n = blockIdx.x;
  L2State st;
  fold_chunk<T, true, kL2RowThreads, kL2RowUnroll>(p, n, 0, st);
  block_merge<kL2RowThreads>(st, 0.f);
  if (threadIdx.x == 0) {
    p.ws_r[n] = st.r;
    p.ws_t[n] = st.t;
    p.out[n] = st.r * __builtin_sqrtf(st.t);
  }
}

// Global nest of the L2 norm: one wave per row combines its chunks (a thread
// per row read them one after another; the two kernels
// took 8.6 us on 69 x 50600 bf16 rows, 5.7 with this and the merges above).
__global__ __launch_bounds__(kNormThreads) void l2_combine_kernel(NormParams p) {
  const int n = blockIdx.x * (kNormThreads / 64) + (threadIdx.x >> 6);
  if (n >= p.N) return;
  const int lane = threadIdx.x & 63;
  L2State st;
  for (int c = lane; c < p.chunks; c += 64)
    st.merge(p.ws_r[(size_t)n * p.chunks + c], p.ws_t[(size_t)n * p.chunks + c], 0.f);
  st.wave_merge(0.f);
  if (lane == 0) p.out[n] = st.r * __builtin_sqrtf(st.t);
}

template <typename T>
__device__ __forceinline__ u32x4 scaled(const u32x4& w, float q) {
  constexpr int VN = Vec<T>::N;
  float f[VN];
  Vec<T>::load(w, f);
#pragma unroll
  for (int k = 0; k < VN; ++k) f[k] *= q;
  return Vec<T>::store(f);
}

// RMSNorm output: every workgroup (chunk c, row n) combines its row's
// partials (s = the row mean of x^2, m = the row max of y), writes m if it
// holds chunk 0, and writes its chunk of y = x / sqrt(s + eps).
template <typename T>
__global__ __launch_bounds__(kNormThreads) void rms_apply_kernel(NormParams p) {
  constexpr int VN = Vec<T>::N;
  const int c = blockIdx.x % p.chunks, n = blockIdx.x / p.chunks;
  __shared__ float s_q;
  if (threadIdx.x < 64) {
    RmsState st;
    for (int k = threadIdx.x; k < p.chunks; k += 64)
      st.merge(p.ws_r[(size_t)n * p.chunks + k], p.ws_t[(size_t)n * p.chunks + k], p.eps);
    st.wave_merge(p.eps);
    if (threadIdx.x == 0) {
      s_q = 1.f / __builtin_sqrtf(st.r + p.eps);
      if (c == 0) p.out[n] = st.t;
    }
  }
  __syncthreads();
  const float q = s_q;
  const int v0 = (int)(min((long long)c * p.chunk, (long long)p.M) / VN);
  const int v1 = (int)(min((long long)(c + 1) * p.chunk, (long long)p.M) / VN);
  const u32x4* row = reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(p.x) + (size_t)n * p.M);
  u32x4* yrow = reinterpret_cast<u32x4*>(reinterpret_cast<T*>(p.y) + (size_t)n * p.M);
  auto batch = [&](auto kc, int b) {
    constexpr int K = decltype(kc)::value;
    u32x4 w[K];
#pragma unroll
    for (int u = 0; u < K; ++u) w[u] = load16<true>(row + min(b + (int)threadIdx.x + u * kNormThreads, v1 - 1));
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const int v = b + (int)threadIdx.x + u * kNormThreads;
      if (v < v1) __builtin_nontemporal_store(scaled<T>(w[u], q), yrow + v);
    }
  };
  int b = v0;
  for (; v1 - b > kNormThreads; b += kApplyUnroll * kNormThreads)
    batch(std::integral_constant<int, kApplyUnroll>{}, b);
  if (b < v1) batch(std::integral_constant<int, 1>{}, b);
}

// The row max of y from the row max of x and r = the mean square: m / sqrt(r +
// eps), as the rolling state ends up: 0 where r has overflowed, -inf where
// there is no scale (r + eps = 0).
__device__ __forceinline__ float rms_rowmax(float m, float r, float eps, float q) {
  const float d = r + eps;
  if (d == 0.f || m == kNegInf) return kNegInf;
  return d == -kNegInf ? 0.f : m * q;
}

// Keep the loaded words, not their conversions, live until the stores (half
// the registers for fp16 and bf16).
__device__ __forceinline__ void keep_words(u32x4& w) { asm volatile("" : "+v"(w)); }

// One-pass RMSNorm.  The row is held in registers, so the producer is known
// before the consumer needs it: the lanes reduce r (the mean square) and the
// plain max, h is applied once, and y is written from the registers.
template <typename T, int V, int RW>
__device__ __forceinline__ void rms_wave_rows(const NormParams& p, int nv) {
  const int lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6)) * RW;
  if (n0 >= p.N) return;
  u32x4 w[RW][V];
  load_rows<T, V, RW>(p, n0, nv, w);
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    float r = 0.f, m = kNegInf;
    RmsState::sums<T, V>(w[i], [&](int u) { return lane + 64 * u < nv; }, p.invM, r, m);
#pragma unroll
    for (int u = 0; u < V; ++u) keep_words(w[i][u]);
    r = wave_sum(r);
    m = wave_max(m);
    const int n = n0 + i;
    if (n >= p.N) break;
    const float q = 1.f / __builtin_sqrtf(r + p.eps);
    if (lane == 0) {
      const float t = rms_rowmax(m, r, p.eps, q);
      p.ws_r[n] = r;
      p.ws_t[n] = t;
      p.out[n] = t;
    }
    u32x4* yrow = reinterpret_cast<u32x4*>(p.y) + (size_t)n * nv;
#pragma unroll
    for (int u = 0; u < V; ++u)
      if (lane + 64 * u < nv) yrow[lane + 64 * u] = scaled<T>(w[i][u], q);
  }
}

// One workgroup (of blockDim.x lanes) per row of at most blockDim.x V vectors,
// read in batches of BATCH vectors a lane, each folded before the next is
// issued (the empty asm with a memory clobber keeps the next batch's loads
// after the fold).
template <typename T, int V, int BATCH>
__device__ __forceinline__ void rms_block_row(const NormParams& p, int nv) {
  const int n = blockIdx.x, nth = blockDim.x;
  const u32x4* row = reinterpret_cast<const u32x4*>(p.x) + (size_t)n * nv;
  u32x4 w[V];
  float r = 0.f, m = kNegInf;
#pragma unroll
  for (int b0 = 0; b0 < V; b0 += BATCH) {
    if (b0 * nth >= nv) break;
#pragma unroll
    for (int u = b0; u < b0 + BATCH; ++u) w[u] = load16<true>(row + min((int)threadIdx.x + u * nth, nv - 1));
    RmsState::sums<T, BATCH>(w + b0, [&](int u) { return (int)threadIdx.x + (b0 + u) * nth < nv; }, p.invM, r, m);
#pragma unroll
    for (int u = b0; u < b0 + BATCH; ++u) keep_words(w[u]);
    if (V > BATCH) asm volatile("" ::: "memory");
  }
  __shared__ float sr[kRowThreads / 64], sm[kRowThreads / 64];
  r = wave_sum(r);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) {
    sr[threadIdx.x >> 6] = r;
    sm[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  r = sr[0];
  m = sm[0];
  for (int k = 1; k < nth / 64; ++k) {
    r += sr[k];
    m = fmaxf(m, sm[k]);
  }
  const float q = 1.f / __builtin_sqrtf(r + p.eps);
  if (threadIdx.x == 0) {
    const float t = rms_rowmax(m, r, p.eps, q);
    p.ws_r[n] = r;
    p.ws_t[n] = t;
    p.out[n] = t;
  }
  u32x4* yrow = reinterpret_cast<u32x4*>(p.y) + (size_t)n * nv;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int v = (int)threadIdx.x + u * nth;
    if (v < nv) yrow[v] = scaled<T>(w[u], q);
  }
}

// HBM-bound: X is read and y written once (256 x 2^17 bf16: 21.8 us, 6.15
// TB/s).  p.lanes lanes per row (see rms_row_lanes).  With 1024 lanes and 16
// vectors each, 2 vectors a lane are in flight at a time, 32 KiB per workgroup:
// when the lanes' sums were still folded vector by vector, 5.33 TB/s on those
// rows against 4.78 with the whole row in flight at once (4 a batch: 5.13; 1:
// 5.03).
template <typename T>
__global__ __launch_bounds__(kRowThreads) void rms_row_kernel(NormParams p) {
  const int nv = p.M / Vec<T>::N;
  if (p.lanes == 64) {
    if (nv <= 64) rms_wave_rows<T, 1, 1>(p, nv);
    else if (nv <= 128) rms_wave_rows<T, 2, 1>(p, nv);
    else if (nv <= 256) rms_wave_rows<T, 4, 1>(p, nv);
    else rms_wave_rows<T, 8, 1>(p, nv);
  } else if (nv <= 4 * p.lanes) {
    rms_block_row<T, 4, 4>(p, nv);
  } else if (p.lanes < kRowThreads) {
    rms_block_row<T, kRowVecs, kShareBatch>(p, nv);
  } else {
    rms_block_row<T, kRowVecs, kRowBatch>(p, nv);
  }
}

// Lanes per row of the one-pass RMSNorm, by the row's vectors.  Short rows: a
// wave each, all loads in flight, no barrier (2048 x 4096 bf16: 7.4 us, 8.4
// with a workgroup a row, 47.8 with 1024 lanes whatever the row).  Longer
// ones: four vectors a lane.  Past 2048 vectors a workgroup wide enough for
// that is alone on its compute unit, and its reads and writes alternate; with
// a row for every compute unit, 16 vectors a lane let 2 to 5 rows share it
// (700 x 20000 bf16: 10.2 us against 14.6; 1000 x 32768: 22.1 against 29.2),
// with fewer rows the wide one finishes a row sooner (64 x 32768: 4.1 us).
int rms_row_lanes(int N, int nv) {
  if (nv <= kWaveRowVecs) return 64;
  if (nv <= 4 * 256) return 256;
  if (nv <= 4 * 512) return 512;
  if (N >= kRowsToShare && nv <= kRowVecs * 256) return 256;
  if (N >= kRowsToShare && nv <= kRowVecs * 512) return 512;
  return kRowThreads;
}

template <typename T>
hipError_t launch_norm_t(const NormParams& p, hipStream_t stream) {
  const dim3 grid(p.N * p.chunks), block(kNormThreads);
  if (norm_one_kernel(p.rms != 0, p.M, (int)sizeof(T), p.chunks)) {
    const int nv = p.M / Vec<T>::N;
    NormParams q = p;
    q.lanes = p.rms ? rms_row_lanes(p.N, nv) : nv <= kWaveRowVecs ? 64 : kL2RowThreads;
    const int rpw = q.lanes == 64 ? kNormThreads / 64 : 1;   // rows per workgroup
    const dim3 rgrid((p.N + rpw - 1) / rpw), rblock(q.lanes == 64 ? kNormThreads : q.lanes);
    if (p.rms)
      hipLaunchKernelGGL((rms_row_kernel<T>), rgrid, rblock, 0, stream, q);
    else
      hipLaunchKernelGGL((l2_row_kernel<T>), rgrid, rblock, 0, stream, q);
    return hipGetLastError();
  }
  if (p.rms) {
    hipLaunchKernelGGL((norm_split_kernel<T, true>), grid, block, 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rms_apply_kernel<T>), grid, block, 0, stream, p);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((norm_split_kernel<T, false>), grid, block, 0, stream, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(l2_combine_kernel, dim3((p.N + kNormThreads / 64 - 1) / (kNormThreads / 64)), block,
                     0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_norm(const NormParams& p, hipStream_t stream) {
  if (p.dtype == 2) return launch_norm_t<float>(p, stream);
  return p.dtype == 1 ? launch_norm_t<__bf16>(p, stream) : launch_norm_t<_Float16>(p, stream);
}

}  // namespace attn
