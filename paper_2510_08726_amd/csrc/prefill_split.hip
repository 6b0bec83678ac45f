// Prefill for few query rows: the rolling update of prefill.hip with each
// item's keys split inside the workgroup (split-k update, Section "Split-K
// Update", Fig. su-result, with the global nests run through LDS).
//
// prefill.hip gives a wave 32 query rows and all their keys, four such waves a
// workgroup.  A short prompt, or a piece of a long one against its cache, has
// too few rows to give every compute unit such a workgroup (1 x 32/8 heads, 64
// rows: 16 workgroups), and the key loop of each is a serial chain.  Here a
// workgroup has 8 waves: G key groups, each with its share of the item's key
// tiles, times 8 / G column blocks of 32 (query row, head) columns that share
// their group's tiles.  The groups' (O, max, sum) are merged through LDS at
// the end.  With a workspace an item's keys are also divided over workgroups
// (p.splits ranges), whose merged partials prefill_combine_kernel combines.
//
// Per tile of 32 keys a wave computes S^T = K . Q^T (32 keys x 32 columns), the
// online softmax per column (lane pair), and O^T += V^T . P^T, with the operand
// layouts of decode.hip.  K and V tiles pass through kStages LDS buffers per
// group, filled by buffer loads that write LDS directly.
//
// What bounds it: the step of a workgroup, not one unit.  With 4 groups (D =
// 128) a step reads 64 KB of tiles while the next 64 KB are on their way, and
// takes 1.2 us: about 55 GB/s for a compute unit, from past its XCD's L2.  Every
// group waits for its copies with nothing else in flight, and at a barrier for
// the slowest group.  Counters (1 x 32/8 heads, 500 rows on 6100 keys): MFMA
// busy 0.30 of the SIMD cycles, VALU active 0.29; of a wave's cycles 0.36 wait
// for copies, barriers and results, 0.32 for issue, 0.32 issue.  (Touching later
// tiles ahead of their copies was 10 % slower.)  With 2 groups, four buffers and
// three tiles in flight each, the two waves of a SIMD take 0.95 us.  Hence the
// choice between more groups (fewer steps) and more columns per tile fetched,
// and the key ranges over more compute units: see the plan below.

#include <algorithm>
#include <cmath>

#include "kernel_common.h"
#include "launch.h"

namespace attn {

namespace {

constexpr int kWaves = 8;                    // key groups times column blocks of 32
constexpr int kThreads = 64 * kWaves;
constexpr int TN = 32;                       // keys per tile
constexpr int kXcds = 8;
constexpr float kLazyThreshold = 8.f;        // as in prefill.hip (log2 units)
constexpr float kMcInit = -1e30f;            // reference before the first visible key

// LDS buffers (of a K and a V tile) per key group: 128 KB of tiles at D = 128,
// 64 KB at D = 64.
template <int D, int G> constexpr int kStages = G == 2 ? 4 : 2;

__device__ __forceinline__ float max_halves(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned a = r[0], b = r[1];
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}

// 4x4x4 MFMA with an all-ones operand: adds the four 16-bit values that each
// lane holds in b to every register of c, so the exp-sum is accumulated from
// the same rounded weights that multiply V (as in prefill.hip).
template <typename T> struct RowSum;
template <> struct RowSum<_Float16> {
  typedef _Float16 v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ f32x4 add(uint2 b, f32x4 c) {
    const v4 one = {(_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f};
    return __builtin_amdgcn_mfma_f32_4x4x4f16(one, __builtin_bit_cast(v4, b), c, 0, 0, 0);
  }
};
template <> struct RowSum<__bf16> {
  typedef short v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ f32x4 add(uint2 b, f32x4 c) {
    const v4 one = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(one, __builtin_bit_cast(v4, b), c, 0, 0, 0);
  }
};

template <int D, typename T, int G, bool ALIBI, bool CAP>
__global__ __launch_bounds__(kThreads, D == 64 ? 4 : 2) void prefill_split_kernel(PrefillSplitParams p) {
  typedef Elem<T> E;
  typedef typename E::vec8 vec8;
  constexpr bool LOG2 = ALIBI || CAP;          // scores prepared in log2 units before the max
  constexpr int KX = D / 16;                   // MFMA K-steps of K.Q^T
  constexpr int DB = D / 32;                   // 32-dim blocks of O^T
  constexpr int TB = TN * D * (int)sizeof(T);  // bytes of a K or V tile
  constexpr int NBLK = TB / 1024;              // 1 KB copies per tile
  constexpr int CPR = D / 8;                   // 16-byte chunks per row
  constexpr int kGroups = G, kCols = kWaves / G;
  constexpr int NST = kStages<D, G>;
  constexpr int CPW = 2 * NBLK / kCols;        // copies per wave of its group's tile pair
  constexpr int kRing = kGroups * NST * 2 * TB;
  constexpr int kMerge = kGroups * kCols * 32 * D * 4;
  constexpr int kTiles = kRing > kMerge ? kRing : kMerge;
  __shared__ __attribute__((aligned(1024))) char lds[kTiles + kGroups * kCols * 32 * 8];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / kCols, cb = wave % kCols;
  const int n = lane & 31, hh = lane >> 5;

  // Item: an XCD takes a contiguous share (workgroup g runs on XCD g mod 8),
  // so that the readers of a KV head share its L2.
  const int x = blockIdx.x % kXcds;
  const int s0 = (int)((long long)p.nitems * x / kXcds), s1 = (int)((long long)p.nitems * (x + 1) / kXcds);
  const int item = s0 + blockIdx.x / kXcds;
  if (item >= s1) return;
  const int hg = p.hg;                                   // heads per item (a power of two up to kCols)
  const int us = item / p.nqb;
  const int rb = p.nqb - 1 - (item - us * p.nqb);
  const int unit = us / p.splits, sp = us - unit * p.splits;   // key range sp of the item's p.splits
  const int ngrp = p.group / hg;
  const int kvh = unit / ngrp;
  const int head = kvh * p.group + (unit - kvh * ngrp) * hg + cb % hg;
  const int Lq = p.Lq, Lk = p.Lk, off = Lk - Lq, W = p.window;
  const int rows = 32 * (kCols / hg);                    // query rows per item
  const int i0 = rb * rows;
  const int iw = i0 + 32 * (cb / hg);                    // this wave's first row
  // Row i sees keys [lo(i), hi(i)).
  auto hi = [&](int i) { return p.causal ? min(Lk, max(0, i + off + 1)) : Lk; };
  auto lo = [&](int i) { return W > 0 ? min(Lk, max(0, i + off + 1 - W)) : 0; };
  const int ilast = min(i0 + rows, Lq) - 1;
  const int ta = lo(i0) / TN, tb = max(ta, (hi(ilast) + TN - 1) / TN);
  const int ps = (tb - ta + p.splits - 1) / p.splits;
  const int t0 = min(ta + sp * ps, tb), t1 = min(t0 + ps, tb);
  const int per = (t1 - t0 + kGroups - 1) / kGroups;     // tiles per key group: iterations of every wave
  const int g0 = min(t0 + kg * per, t1);
  const int gn = min(per, t1 - g0);                      // this group's tiles
  // This wave's rows see keys in tiles [a, b), and every row sees all keys of
  // tiles [wl, wh).
  const int wlast = min(iw + 32, Lq) - 1;
  int a = 0, b = 0, wl = 0, wh = 0;
  if (iw < Lq && hi(wlast) > lo(iw)) {
    a = lo(iw) / TN;
    b = (hi(wlast) + TN - 1) / TN;
    wl = (lo(wlast) + TN - 1) / TN;
    wh = hi(iw) / TN;
  }
  const int row = min(iw + n, Lq - 1);                   // this lane's row (repeated past the last)
  const int rhi = hi(row), rlo = lo(row);

  // Copies: the group's waves each move CPW of the 1 KB blocks of a tile pair,
  // the first half of them K, the others V, through one buffer resource whose
  // range ends at the head's last key (rows past it read as zero).
  const int kv = cb / (kCols / 2), blk0 = cb % (kCols / 2) * CPW;
  const T* src = reinterpret_cast<const T*>(kv == 0 ? p.k : p.v) + (size_t)kvh * Lk * D;
  const uint64_t sa = reinterpret_cast<uint64_t>(src);
  const u32x4 rsrc = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sa),
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(sa >> 32) & 0xffffu)),
                      (uint32_t)__builtin_amdgcn_readfirstlane(Lk * D * (int)sizeof(T)), 0x00020000u};
  char* const gl = lds + kg * NST * 2 * TB;              // this group's buffers: NST of (K tile, V tile)
  const uint32_t gl_addr = (uint32_t)(uintptr_t)(lds_void*)gl;
  int goff[CPW];
#pragma unroll
  for (int u = 0; u < CPW; ++u) {
    const int r = (blk0 + u) * (1024 / (2 * D)) + lane / CPR;
    const int pos = lane % CPR;
    goff[u] = (r * D + 8 * (pos ^ swz<D>(r))) * (int)sizeof(T);
  }
  auto copy_tile = [&](int t) __attribute__((always_inline)) {   // tile t of the group
    // The tile's offset goes into the lane offset, which the range check covers.
    const int tb = __builtin_amdgcn_readfirstlane((g0 + t) * TB);
    const uint32_t dst = gl_addr + (uint32_t)(((t % NST) * 2 + kv) * TB + blk0 * 1024);
#pragma unroll
    for (int u = 0; u < CPW; ++u)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   : : "s"(dst + (uint32_t)(u * 1024)), "v"(goff[u] + tb), "s"(rsrc) : "memory", "m0");
  };

  // Per-lane LDS offsets of the K and V^T fragments (see decode.hip).
  int ak[KX], av[DB][2];
#pragma unroll
  for (int kx = 0; kx < KX; ++kx) ak[kx] = 2 * (n * D + 8 * ((2 * kx + hh) ^ swz<D>(n)));
  {
    const int Gq = lane >> 4, i = lane & 15;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int lh = 0; lh < 2; ++lh) {
        const int d = 32 * db + 16 * (Gq & 1) + 4 * (i & 3);
        const int k = 4 * (Gq >> 1) + (i >> 2) + 8 * lh;
        av[db][lh] = 2 * (k * D + 8 * ((d >> 3) ^ swz<D>(k)) + (d & 7));
      }
  }

#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < gn) copy_tile(t);

  // Q^T as the B operand: lane (n, hh) holds Q[row][16 kx + 8 hh ..].
  vec8 qf[KX];
  {
    const T* qp = reinterpret_cast<const T*>(p.q) + ((size_t)head * Lq + row) * D + 8 * hh;
#pragma unroll
    for (int kx = 0; kx < KX; ++kx) {
      u32x4 w = *reinterpret_cast<const u32x4*>(qp + 16 * kx);
      if (!LOG2) w ^= p.qsign;
      qf[kx] = __builtin_bit_cast(vec8, w);
    }
  }
  const float c = p.c, k2 = p.cap_k2 * p.c, cl = p.cap_cl;
  const float ce = LOG2 ? 1.f : c;
  const float sl2 = ALIBI ? p.slopes[head % p.Hq] * kLog2e : 0.f;

  float mc = kMcInit;               // reference (log2 units)
  f32x4 l4 = {0.f, 0.f, 0.f, 0.f};  // this lane's half of the exp-sum, four times
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = f32x16{};

  for (int t = 0; t < per; ++t) {
    // Tile t is in LDS when every wave of the group has waited for its own
    // copies; the buffer of tile t - 1, whose reads every wave has waited
    // for, is free behind the same barrier.
    if (t + NST - 2 < gn)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((NST - 2) * CPW) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (t + NST - 1 < gn) copy_tile(t + NST - 1);
    const int tile = g0 + t;
    if (t >= gn || tile < a || tile >= b) continue;
    const char* kt = gl + (t % NST) * 2 * TB;
    const char* vt = kt + TB;

    f32x16 s = f32x16{};
#pragma unroll
    for (int kx = 0; kx < KX; ++kx) {
      const vec8 kf = __builtin_bit_cast(vec8, *reinterpret_cast<const u32x4*>(kt + ak[kx]));
      s = E::mfma(kf, qf[kx], s);
    }
    // Register r of lane (n, hh) is key 8 (r / 4) + 4 hh + r % 4 of the tile.
    const int j0 = tile * TN + 4 * hh;
    if (LOG2) {
      const float base = ALIBI ? sl2 * (float)(j0 - iw - off) : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float kc = (float)(8 * (r / 4) + r % 4);
        if (CAP) s[r] = soft_cap(s[r], k2, cl);
        else s[r] = __builtin_fmaf(s[r], c, __builtin_fmaf(sl2, kc, base));
      }
    }
    if (tile < wl || tile >= wh) {
      const int lh = rhi - j0, ll = rlo - j0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int kc = 8 * (r / 4) + r % 4;
        s[r] = (kc < lh && kc >= ll) ? s[r] : kNegInf;
      }
    }
    float tm = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s[r]);
    tm = max_halves(tm);
    // Lazy repair: the reference moves when the row's maximum exceeds it by
    // more than the threshold (always at the row's first visible key).
    const float d = __builtin_fmaf(tm, ce, -mc);
    if (__builtin_amdgcn_ballot_w64(d > kLazyThreshold) != 0) {
      const bool move = d > kLazyThreshold;
      const float alpha = move ? fast_exp2(-d) : 1.f;
      mc = move ? tm * ce : mc;
      l4 *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] *= alpha;
    }
    uint32_t w[2][4];
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const float p0 = fast_exp2(__builtin_fmaf(s[r], ce, -mc));
      const float p1 = fast_exp2(__builtin_fmaf(s[r + 1], ce, -mc));
      w[r / 8][(r % 8) / 2] = E::pack2(p0, p1);
    }
#pragma unroll
    for (int c16 = 0; c16 < 2; ++c16)
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) l4 = RowSum<T>::add(make_uint2(w[c16][2 * h2], w[c16][2 * h2 + 1]), l4);
#pragma unroll
    for (int c16 = 0; c16 < 2; ++c16) {
      const vec8 pb = __builtin_bit_cast(vec8, make_uint4(w[c16][0], w[c16][1], w[c16][2], w[c16][3]));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const char* base = vt + c16 * 32 * D;
        const uint2 vlo = lds_read_tr(base + av[db][0]);
        const uint2 vhi = lds_read_tr(base + av[db][1]);
        const vec8 vf = __builtin_bit_cast(vec8, make_uint4(vlo.x, vlo.y, vhi.x, vhi.y));
        o[db] = E::mfma(vf, pb, o[db]);
      }
    }
  }

  // Merge the key groups through LDS (the tile buffers are free after the
  // barrier).  Lane (n, hh) holds O^T[32 db + 8 i + 4 hh + j][column n] in
  // register 4 i + j of block db: 16-byte chunk 8 db + 2 i + hh of the
  // column's row, stored at chunk ^ (n mod 16) so that neighbouring columns
  // use different banks.
  __syncthreads();
  float* sh_o = reinterpret_cast<float*>(lds);                         // [wave][32][D]
  float* sh_m = reinterpret_cast<float*>(lds + kTiles);                // [wave][32]
  float* sh_l = sh_m + kGroups * kCols * 32;                           // [wave][32]
  const float l = l4[0] + swap_halves(l4[0]);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ch = (8 * db + 2 * i + hh) ^ (n & 15);
      const f32x4 v = {o[db][4 * i], o[db][4 * i + 1], o[db][4 * i + 2], o[db][4 * i + 3]};
      *reinterpret_cast<f32x4*>(sh_o + (wave * 32 + n) * D + 4 * ch) = v;
    }
  if (hh == 0) {
    sh_m[wave * 32 + n] = mc;
    sh_l[wave * 32 + n] = l;
  }
  __syncthreads();
  // Column block cb's waves write its rows: each thread whole 16-byte chunks,
  // D / 4 neighbouring threads a row.
  const int ct = kg * 64 + lane;                                       // thread within the column block
  T* op = reinterpret_cast<T*>(p.o) + ((size_t)head * Lq + iw) * D;
  constexpr int CH = D / 4;
#pragma unroll 1
  for (int u = 0; u < 32 * CH / (64 * kGroups); ++u) {
    const int idx = u * 64 * kGroups + ct;
    const int col = idx / CH, ch = idx % CH;
    float M = kMcInit;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) M = fmaxf(M, sh_m[(g * kCols + cb) * 32 + col]);
    float L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      const int wv = g * kCols + cb;
      const float f = fast_exp2(sh_m[wv * 32 + col] - M);
      L = __builtin_fmaf(sh_l[wv * 32 + col], f, L);
      acc += f * *reinterpret_cast<const f32x4*>(sh_o + (wv * 32 + col) * D + 4 * (ch ^ (col & 15)));
    }
    if (p.splits > 1) {
      // A key range's partial, in log2 units; the combine kernel follows.
      if (iw + col < Lq) {
        const size_t nr = (size_t)p.nheads * Lq, r = sp * nr + (size_t)head * Lq + iw + col;
        *reinterpret_cast<f32x4*>(p.ws + r * D + 4 * ch) = acc;
        if (ch == 0) *reinterpret_cast<float2*>(p.ws + p.splits * nr * D + 2 * r) = make_float2(M, L);
      }
      continue;
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    uint2 out;
    out.x = E::pack2(acc[0] * inv, acc[1] * inv);
    out.y = E::pack2(acc[2] * inv, acc[3] * inv);
    if (iw + col < Lq) *reinterpret_cast<uint2*>(op + (size_t)col * D + 4 * ch) = out;
  }
}

// Global nests over the key ranges: D / 4 threads a row, kBatch ranges' loads
// in flight at a time.
template <int D, typename T>
__global__ __launch_bounds__(256) void prefill_combine_kernel(PrefillSplitParams p) {
  constexpr int kBatch = 8, CH = D / 4;
  const size_t nr = (size_t)p.nheads * p.Lq;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t row = idx / CH;
  const int ch = (int)(idx % CH);
  if (row >= nr) return;
  const float* ml = p.ws + p.splits * nr * D;
  float M = kMcInit, L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < p.splits; s0 += kBatch) {
    f32x4 v[kBatch];
    float2 w[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {   // past the last range: that range again, left out below
      const size_t r = min(s0 + u, p.splits - 1) * nr + row;
      v[u] = *reinterpret_cast<const f32x4*>(p.ws + r * D + 4 * ch);
      w[u] = *reinterpret_cast<const float2*>(ml + 2 * r);
    }
    float mn = M;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) mn = fmaxf(mn, w[u].x);
    const float a = fast_exp2(M - mn);
    L *= a;
    acc *= a;
    M = mn;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      // (By its values, not by its weight: 0 times an infinite value would be NaN.)
      const bool in = s0 + u < p.splits;
      const float f = in ? fast_exp2(w[u].x - mn) : 0.f;
      L = __builtin_fmaf(w[u].y, f, L);
      acc += f * (in ? v[u] : f32x4{0.f, 0.f, 0.f, 0.f});
    }
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;
  uint2 out;
  out.x = Elem<T>::pack2(acc[0] * inv, acc[1] * inv);
  out.y = Elem<T>::pack2(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<uint2*>(reinterpret_cast<T*>(p.o) + row * D + 4 * ch) = out;
}

template <int D, typename T, int G>
void launch_g(const PrefillSplitParams& p, hipStream_t stream) {
  const dim3 grid((p.nitems + kXcds - 1) / kXcds * kXcds), block(kThreads);
  if (p.slopes) hipLaunchKernelGGL((prefill_split_kernel<D, T, G, true, false>), grid, block, 0, stream, p);
  else if (p.cap_cl != 0.f) hipLaunchKernelGGL((prefill_split_kernel<D, T, G, false, true>), grid, block, 0, stream, p);
  else hipLaunchKernelGGL((prefill_split_kernel<D, T, G, false, false>), grid, block, 0, stream, p);
}

template <int D, typename T>
hipError_t launch_d(const PrefillSplitParams& p, int kgroups, hipStream_t stream) {
  if (kgroups == 2) launch_g<D, T, 2>(p, stream);
  else launch_g<D, T, 4>(p, stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.splits == 1) return e;
  const size_t threads = (size_t)p.nheads * p.Lq * (D / 4);
  hipLaunchKernelGGL((prefill_combine_kernel<D, T>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

// Heads and row blocks of one item with c column blocks: as many heads of a
// KV head as divide the group (they share its tiles), the rest rows.
int heads_per_item(int group, int c) {
  int hg = 1;
  while (hg < c && group % (2 * hg) == 0) hg *= 2;
  return hg;
}
int64_t items_of(int B, int Hq, int group, int Lq, int c) {
  const int hg = heads_per_item(group, c), rows = 32 * (c / hg);
  return (int64_t)((Lq + rows - 1) / rows) * ((int64_t)B * Hq / hg);
}

// Which kernel, how many key groups a workgroup and how many key ranges over
// workgroups: the least estimated time.  The estimates are linear in the tiles
// of the longest item, in us, and fitted to 4000 random shapes that give
// prefill.hip at most 256 workgroups, under all plans (1 to 5000 rows, up to
// 20000 keys, both head dims, every modifier); nine in ten are within 12 %.
// prefill.hip: a start and end, longer with a window or ALiBi, and a cost for a
// tile, larger with a cap.  Here: a start and end, the first tiles (each key
// group in use starts another fetch) and a cost for an iteration, taken
// between the whole iterations and the tiles' share of them.  Where the
// workgroups outnumber the compute units:
//  - D = 128 (a workgroup takes a compute unit's LDS) starts the others as the
//    first end, within each XCD's share of the items: the longest of them, and
//    a start and end more (several ranges go there only where even two of the
//    fewest items don't fit one round);
//  - D = 64 runs two at a time, which share the compute unit's fetches: the
//    items of a compute unit one after another, half of a last incomplete
//    round where they are alike.
// Several key ranges cost the combine kernel, one latency for 8 of them, and
// the partials' way through memory.  The split has to win by 4 %: on those
// shapes the kernel taken is then never more than 3 % behind prefill.hip, and
// on average 0.6 % behind the best of all.
// Measured, prefill.hip and here: 1 x 32/8 heads, 500 rows on 6100 keys 93 and
// 64 us (4 groups, 1 range); 64 on 16000 230 and 31 (4, 8); 2 x 32/16, 130 on
// 13392 197 and 115 (2, 2); D = 64, 1 x 32/4, 200 on 9000 100 and 34 (4, 2); 1 x
// 32 x 482 14.5 and 12.0 (4, 1); but 6 x 8 x 361 12.9 and 17.4 (4, 1), and D =
// 64, 4 x 2 x 8 5.0 and 5.3 (4, 1).
PrefillSplitPlan prefill_split_plan(int B, int Hq, int Hkv, int Lq, int Lk, int D, bool causal, int window, bool alibi,
                                    bool cap, int cus, int max_splits) {
  const int group = Hq / Hkv;
  const int64_t wide = items_of(B, Hq, group, Lq, 4);   // workgroups of prefill.hip
  if (wide > cus) return {0, 1};
  // Keys of the longest, the average and the lightest item with c column
  // blocks; `grow` of a unit's items see fewer keys than the one before.
  struct Keys {
    float most, mean, light, grow;
    // Keys of the item at the fraction f of a unit, heaviest first.
    float at(float f) const { return f <= 1.f - grow ? most : light + (most - light) * std::max(0.f, 1.f - f) / grow; }
  };
  auto keys = [&](int c) {
    Keys k = {(float)Lk, 0.f, (float)Lk, 0.f};
    if (causal) {
      k.light = std::max(0.f, (float)Lk - Lq);
      k.grow = 1.f;
    }
    if (window > 0) {
      k.most = std::min(k.most, (float)window + 32 * (c / heads_per_item(group, c)));
      k.light = std::min(k.light, k.most);
      k.grow = std::min(1.f, std::max(0.f, (float)window - ((float)Lk - Lq)) / Lq);
    }
    k.mean = k.most - 0.5f * k.grow * (k.most - k.light);
    return k;
  };
  // By head dim: 64, 128.
  struct Split { float start, first, iter[3]; };   // iter: plain, ALiBi, SoftCap
  static constexpr Split kSplit[2][2] = {{{4.55f, 0.67f, {0.72f, 0.89f, 1.13f}}, {5.45f, 1.42f, {1.16f, 1.32f, 1.39f}}},
                                         {{4.85f, 0.51f, {0.69f, 0.83f, 1.04f}}, {5.95f, 1.13f, {1.00f, 1.15f, 1.25f}}}};
  struct Wide { float start, window, alibi, alibi_all, tile, tile_window, tile_alibi, tile_cap; };
  static constexpr Wide kWide[2] = {{4.95f, 1.55f, 1.1f, 0.8f, 0.366f, 0.045f, 0.035f, 0.16f},
                                    {5.85f, 3.6f, 2.8f, 1.7f, 0.492f, 0.07f, 0.045f, 0.15f}};
  const int d = D == 128;
  auto best = [&](bool alibi, bool cap, int max_splits) {
    const Wide& w = kWide[d];
    const float start = w.start + (window > 0 ? w.window : !alibi ? 0.f : causal ? w.alibi : w.alibi_all);
    const float tile = w.tile + (cap ? w.tile_cap : alibi ? w.tile_alibi : 0.f) + (window > 0 ? w.tile_window : 0.f);
    float least = 0.96f * (start + tile * std::ceil(keys(4).most / TN));
    PrefillSplitPlan plan = {0, 1};
    for (int G : {4, 2}) {
      const Split& c = kSplit[G == 2][d];
      const float iter = c.iter[cap ? 2 : alibi ? 1 : 0];
      const int64_t items = items_of(B, Hq, group, Lq, kWaves / G);
      const Keys k = keys(kWaves / G);
      const float alike = k.light / k.most;
      const float unit = (float)items / ((int64_t)B * Hq / heads_per_item(group, kWaves / G));   // items of a unit
      for (int S = 1; S <= max_splits; ++S) {
        const int64_t n = items * S;
        if (d && n > (S > 1 && 2 * wide <= cus ? cus : 2 * cus)) break;
        const float tiles = std::ceil(k.most / TN / S), whole = std::ceil(tiles / G);
        const float begin = c.start + c.first * (std::min(tiles, (float)G) - 1.f) / (G - 1);
        float t;
        if (n > cus && !d) {
          const float rounds = (float)n / cus;
          const float per = rounds + 0.25f * (1.f - alike) + 0.5f * alike * (std::ceil(rounds) - rounds);
          t = begin + iter * std::max(whole, per * (k.mean / TN / S / G + 0.8f)) + 1.f;
        } else {
          t = begin + iter * 0.5f * (whole + std::max(tiles / G, 1.f));
        }
        if (n > cus && d) {
          // A share of n / 8 items on cus / 8 compute units: `more` of them wait.
          const float more = (float)(n - cus) / kXcds, own = (float)cus / kXcds;
          float two;                                     // keys of the waiting item and the one before it
          if (S > 1) two = k.light + k.most;
          else if (more + own < unit) two = 2.f * k.at(own / unit);   // the share is a part of one unit
          else two = k.light + (more >= unit ? k.most + (k.most - k.light) * (more - unit) / own : k.at(1.f - more / unit));
          t = std::max(t, begin + 7.5f + iter * two / TN / S / G);
        }
        if (S > 1) {
          t += 1.1f + 0.8f * ((S + 7) / 8) + (float)((int64_t)B * Hq * Lq) * S * (D + 2) * 8.f * 0.385e-6f;
          t *= 1.02f;                                    // one range where there is next to nothing between them
        }
        if (t < least) {
          least = t;
          plan = {G, S};
        }
      }
    }
    return plan;
  };
  // attn_fwd_num_splits, which sizes the workspace, knows no modifiers: they
  // choose only among the plans with one range.
  const PrefillSplitPlan plan = best(false, false, max_splits);
  return plan.splits == 1 && (alibi || cap) ? best(alibi, cap, 1) : plan;
}

hipError_t launch_prefill_split(const PrefillSplitParams& p, int kgroups, hipStream_t stream) {
  PrefillSplitParams q = p;
  q.hg = heads_per_item(p.group, kWaves / kgroups);
  const int rows = 32 * (kWaves / kgroups / q.hg);
  q.nqb = (p.Lq + rows - 1) / rows;
  q.nheads = p.B * p.Hq;
  q.nitems = q.nqb * (q.nheads / q.hg) * q.splits;
  if (p.D == 64) return p.bf16 ? launch_d<64, __bf16>(q, kgroups, stream) : launch_d<64, _Float16>(q, kgroups, stream);
  return p.bf16 ? launch_d<128, __bf16>(q, kgroups, stream) : launch_d<128, _Float16>(q, kgroups, stream);
}

}  // namespace attn
