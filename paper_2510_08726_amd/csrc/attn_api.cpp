// C ABI of the fused-attention library: argument validation on the host,
// dispatch to the gfx950 kernels, error reporting.  Every check runs before
// anything is enqueued; the only HIP call among them asks for the current
// device and its compute units, where a workspace's size depends on them.

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>

#include "../../include/attn.h"
#include "../../include/peaks.h"
#include "../../include/norms.h"
#include "launch.h"

namespace {

thread_local int g_last_hip_error = 0;

constexpr float kLog2e = 1.4426950408889634f;
constexpr int64_t kMaxGrid = std::numeric_limits<int32_t>::max();
constexpr int kMinChunk = 256;    // keys per decode chunk chosen by the heuristic (one head per KV head)
constexpr int kMinChunkGrouped = 128;   // grouped heads: at least one 32-key tile per wave
constexpr int kTwoChunks = 1200;        // grouped heads, D = 64: keys per chunk from which two share a compute unit

bool shape_ok(int B, int Hq, int Hkv, int Lq, int Lk) {
  return B >= 1 && Hq >= 1 && Hkv >= 1 && Lq >= 1 && Lk >= 1 && Hq % Hkv == 0;
}

bool dims_supported(int D, attn_dtype dtype) {
  return (D == 64 || D == 128) && (dtype == ATTN_F16 || dtype == ATTN_BF16);
}

// Element counts must stay addressable and the grids within 2^31 - 1 blocks.
bool sizes_fit(int B, int Hq, int Hkv, int Lq, int Lk, int D) {
  const int64_t q = (int64_t)B * Hq * Lq * D;
  const int64_t k = (int64_t)B * Hkv * Lk * D;
  return q < (int64_t(1) << 40) && k < (int64_t(1) << 40);
}

int hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return ATTN_ERR_HIP;
}

// Compute units of the current device, 256 without one (the grouped decode
// kernel wants one workgroup per compute unit: each holds 128 KB of LDS, so
// more would run one after another, each paying its start-up and merge again).
// Looked up once per device: it is asked for on every call that chooses its
// own split.
int compute_units() {
  static std::atomic<int> cached[64];
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
  if (dev < 64 && (n = cached[dev].load(std::memory_order_relaxed)) > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  if (dev < 64) cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

// Query heads that one decode workgroup serves (the grid divides the group by it).
int decode_heads_per_block(int group) {
  const int gh = attn::decode_split_heads(group);
  return gh == 0 ? group : gh;
}

// At most one chunk per `least` keys, at least one chunk.
int clamp_splits(int64_t s, int Lk, int least) {
  return (int)std::max<int64_t>(std::min(s, ((int64_t)Lk + least - 1) / least), 1);
}

// Decode chunks of one workgroup per compute unit: the count below which no
// workspace may fall (attn_decode_num_splits gives as many or more).  The
// grouped kernel's is rounded down: all its workgroups run in one round.
int one_round_splits(int B, int Hq, int Hkv, int Lk, int cus) {
  const int group = Hq / Hkv, gh = attn::decode_split_heads(group);
  if (gh == 0) return clamp_splits(cus / ((int64_t)B * Hkv), Lk, kMinChunkGrouped);
  const int64_t units = (int64_t)B * Hkv * (group / gh);
  return clamp_splits((cus + units - 1) / units, Lk, kMinChunk);
}

const char* dtype_name(attn_dtype dtype) { return dtype == ATTN_BF16 ? "bf16" : "f16"; }

int put(char* buf, size_t len, const char* s) {
  const size_t n = std::strlen(s);
  if (!buf || n + 1 > len) return ATTN_ERR_SHAPE;
  std::memcpy(buf, s, n + 1);
  return ATTN_OK;
}

}  // namespace

extern "C" {

const char* attn_status_string(int status) {
  switch (status) {
    case ATTN_OK: return "ATTN_OK: success";
    case ATTN_ERR_NULL: return "ATTN_ERR_NULL: a required pointer is NULL";
    case ATTN_ERR_SHAPE: return "ATTN_ERR_SHAPE: invalid sizes (need B,Hq,Hkv,Lq,Lk >= 1, Hq % Hkv == 0, num_splits >= 0, window >= 0, finite scale, finite softcap >= 0)";
    case ATTN_ERR_UNSUPPORTED: return "ATTN_ERR_UNSUPPORTED: head dim must be 64 or 128 and dtype ATTN_F16 or ATTN_BF16; softcap and window need the causal mask, softcap excludes ALiBi";
    case ATTN_ERR_WORKSPACE: return "ATTN_ERR_WORKSPACE: workspace too small or not 16-byte aligned (attn_decode_noalloc: the split count needs more than its 16 MiB static workspace)";
    case ATTN_ERR_HIP: return "ATTN_ERR_HIP: a HIP launch failed (see attn_last_hip_error)";
    default: return "unknown attn_status";
  }
}

int attn_last_hip_error(void) { return g_last_hip_error; }

int attn_fwd_num_splits(int B, int Hq, int Hkv, int Lq, int Lk, int D, int causal, int window) {
  if (!shape_ok(B, Hq, Hkv, Lq, Lk) || (D != 64 && D != 128) || window < 0) return 0;
  return attn::prefill_split_plan(B, Hq, Hkv, Lq, Lk, D, causal != 0, window, false, false, compute_units(),
                                  attn::kMaxPrefillSplits).splits;
}

size_t attn_fwd_workspace_bytes(int B, int Hq, int Lq, int D, int num_splits) {
  if (B < 1 || Hq < 1 || Lq < 1 || num_splits < 1 || (D != 64 && D != 128)) return 0;
  if (num_splits == 1) return 0;
  const size_t bytes = (size_t)B * Hq * Lq * num_splits * (size_t)(D + 2) * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}

int attn_fwd_split(const void* Q, const void* K, const void* V, void* O,
                   int B, int Hq, int Hkv, int Lq, int Lk, int D,
                   int causal, float scale, const float* alibi_slopes, float softcap, int window,
                   void* workspace, size_t workspace_bytes, attn_dtype dtype, hipStream_t stream) {
  if (!Q || !K || !V || !O) return ATTN_ERR_NULL;
  if (!shape_ok(B, Hq, Hkv, Lq, Lk) || !std::isfinite(scale)) return ATTN_ERR_SHAPE;
  if (!std::isfinite(softcap) || softcap < 0.f || window < 0) return ATTN_ERR_SHAPE;
  if (!dims_supported(D, dtype)) return ATTN_ERR_UNSUPPORTED;
  if (softcap > 0.f && (!causal || alibi_slopes)) return ATTN_ERR_UNSUPPORTED;
  if (window > 0 && !causal) return ATTN_ERR_UNSUPPORTED;
  if (!sizes_fit(B, Hq, Hkv, Lq, Lk, D)) return ATTN_ERR_SHAPE;
  // The prefill kernel addresses one head's K and V with 32-bit byte offsets.
  if ((int64_t)Lk * D * 2 >= (int64_t(1) << 31)) return ATTN_ERR_SHAPE;
  const int bm = attn::prefill_block_rows();
  const int64_t nqb = ((int64_t)Lq + bm - 1) / bm;
  if (nqb * B * Hq > kMaxGrid) return ATTN_ERR_SHAPE;
  const attn::PrefillSplitPlan plan =
      attn::prefill_split_plan(B, Hq, Hkv, Lq, Lk, D, causal != 0, window, alibi_slopes != nullptr, softcap > 0.f,
                               compute_units(), workspace ? attn::kMaxPrefillSplits : 1);
  const int S = plan.splits;
  if (S > 1 && (workspace_bytes < attn_fwd_workspace_bytes(B, Hq, Lq, D, S) || (reinterpret_cast<uintptr_t>(workspace) & 15)))
    return ATTN_ERR_WORKSPACE;

  attn::PrefillSplitParams p{};
  p.q = Q; p.k = K; p.v = V; p.o = O;
  p.slopes = alibi_slopes;
  p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.Lq = Lq; p.Lk = Lk; p.D = D;
  p.group = Hq / Hkv;
  p.causal = causal != 0;
  p.bf16 = dtype == ATTN_BF16;
  p.cap_k2 = softcap > 0.f ? 2.f / softcap : 0.f;
  p.cap_cl = softcap > 0.f ? softcap * kLog2e : 0.f;
  // A window of Lk keys or more masks nothing, and the kernels' row + Lk - Lq +
  // 1 - window stays within an int.
  p.window = std::min(window, Lk);
  if (alibi_slopes || softcap > 0.f) {
    p.c = scale * kLog2e;
    p.qsign = 0;
  } else {
    // Kept above zero so that masked (-inf) scores times c stay -inf when
    // scale is 0; exp2(s * 1e-30) rounds to exactly 1 for any finite score,
    // the same weights as c = 0.
    p.c = std::fmax(std::fabs(scale) * kLog2e, 1e-30f);
    p.qsign = std::signbit(scale) ? 0x80008000u : 0u;
  }
  p.nqb = (int)nqb;
  p.splits = S;
  p.ws = static_cast<float*>(workspace);
  hipError_t e = plan.kgroups > 0 ? attn::launch_prefill_split(p, plan.kgroups, stream) : attn::launch_prefill(p, stream);
  return e == hipSuccess ? ATTN_OK : hip_fail(e);
}

int attn_fwd_mod(const void* Q, const void* K, const void* V, void* O,
                 int B, int Hq, int Hkv, int Lq, int Lk, int D,
                 int causal, float scale, const float* alibi_slopes, float softcap, int window,
                 attn_dtype dtype, hipStream_t stream) {
  return attn_fwd_split(Q, K, V, O, B, Hq, Hkv, Lq, Lk, D, causal, scale, alibi_slopes, softcap, window, nullptr, 0,
                        dtype, stream);
}

int attn_fwd(const void* Q, const void* K, const void* V, void* O,
             int B, int Hq, int Hkv, int Lq, int Lk, int D,
             int causal, float scale, const float* alibi_slopes,
             attn_dtype dtype, hipStream_t stream) {
  return attn_fwd_mod(Q, K, V, O, B, Hq, Hkv, Lq, Lk, D, causal, scale, alibi_slopes, 0.f, 0, dtype, stream);
}

int attn_decode_num_splits(int B, int Hq, int Hkv, int Lk, int D) {
  if (!shape_ok(B, Hq, Hkv, 1, Lk) || (D != 64 && D != 128)) return 0;
  const int group = Hq / Hkv, cus = compute_units();
  if (group >= 2 && group <= 32) {
    // The grouped kernel: one workgroup per (chunk, KV head, batch).  At D =
    // 128 its LDS (128 KB) lets one run at a time per compute unit, so the most
    // chunks that still run in one round: 6 x 64/8 heads, 4050 keys took 41 us
    // in 6 chunks (288 workgroups), 29 in 5; 13 x 32/8, 20000 keys 230 in 3 and
    // 170 in 2; 11 x 32/16, 3000 keys 63 in 2 and 53 in 1.
    const int one = one_round_splits(B, Hq, Hkv, Lk, cus);
    // At D = 64 two run at a time, and one alone reads at about half their
    // rate: up to two per compute unit, where their chunks are long enough to
    // pay for more partials.  11 x 24/12 heads, 12222 keys took 134 us in 1
    // chunk, 88 in 2; 92 KV heads, 15487 keys 99 us in 2, 79 in 3 and 63 in 5;
    // but 16 KV heads, 4856 keys 13.0 in 16 and 13.4 in 32.
    if (D == 64 && Lk / one >= kTwoChunks) return clamp_splits(2 * cus / ((int64_t)B * Hkv), Lk, kMinChunkGrouped);
    return one;
  }
  // The per-head kernel: one workgroup per compute unit where the heads divide
  // them evenly (measured at steady clock with nontemporal K/V loads, batch
  // 1-32, 2048-32768 keys, D 64 and 128: 2-4 % ahead of two per compute unit
  // on four of five shapes, 1 % behind on the fifth), else up to two, which
  // leaves no compute unit a second chunk alone: 9 x 16 heads (D = 64), 8260
  // keys took 69 us in 2 chunks and 51 in 3, 3 x 32, 2280 keys 25.6 in 3 and
  // 23.7 in 5, 5 x 12 (D = 64), 9942 keys 32 in 5 and 28 in 8.
  const int64_t units = (int64_t)B * Hkv * (group / decode_heads_per_block(group));
  return clamp_splits(cus % units == 0 || units > cus ? (cus + units - 1) / units : 2 * cus / units, Lk, kMinChunk);
}

size_t attn_decode_workspace_bytes(int B, int Hq, int D, int num_splits) {
  if (B < 1 || Hq < 1 || num_splits < 1 || (D != 64 && D != 128)) return 0;
  const size_t n = (size_t)B * Hq * num_splits;
  const size_t bytes = n * (size_t)(D + 2) * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}

}  // extern "C"

namespace {

// Argument checks of the decode entry points (everything but the workspace);
// on success *S is the resolved chunk count.
int decode_check(const void* Q, const void* K, const void* V, void* O, int B, int Hq, int Hkv, int Lk, int D,
                 float scale, float softcap, int num_splits, attn_dtype dtype, int* S) {
  if (!Q || !K || !V || !O) return ATTN_ERR_NULL;
  if (!shape_ok(B, Hq, Hkv, 1, Lk) || num_splits < 0 || !std::isfinite(scale)) return ATTN_ERR_SHAPE;
  if (!std::isfinite(softcap) || softcap < 0.f) return ATTN_ERR_SHAPE;
  if (!dims_supported(D, dtype)) return ATTN_ERR_UNSUPPORTED;
  if (!sizes_fit(B, Hq, Hkv, 1, Lk, D)) return ATTN_ERR_SHAPE;
  *S = num_splits ? num_splits : attn_decode_num_splits(B, Hq, Hkv, Lk, D);
  const int group = Hq / Hkv;
  const int64_t nblocks = (int64_t)*S * (group / decode_heads_per_block(group)) * Hkv * B;
  if (nblocks > kMaxGrid || (int64_t)B * Hq > kMaxGrid) return ATTN_ERR_SHAPE;
  return ATTN_OK;
}

// Launch the split and combine kernels with a checked workspace.
int decode_launch(const void* Q, const void* K, const void* V, void* O, int B, int Hq, int Hkv, int Lk, int D,
                  float scale, const float* alibi_slopes, float softcap, int S, void* workspace, attn_dtype dtype,
                  hipStream_t stream) {
  attn::DecodeParams p{};
  p.q = Q; p.k = K; p.v = V; p.o = O;
  p.slopes = alibi_slopes;
  const size_t n = (size_t)B * Hq * S;
  p.ws_o = static_cast<float*>(workspace);
  p.ws_m = p.ws_o + n * D;
  p.ws_l = p.ws_m + n;
  p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.Lk = Lk; p.D = D;
  p.group = Hq / Hkv;
  p.splits = S;
  p.chunk = (Lk + S - 1) / S;
  p.bf16 = dtype == ATTN_BF16;
  p.c = scale * kLog2e;
  p.cap_k2 = softcap > 0.f ? 2.f / softcap : 0.f;
  p.cap_cl = softcap > 0.f ? softcap * kLog2e : 0.f;
  hipError_t e = attn::launch_decode(p, stream);
  return e == hipSuccess ? ATTN_OK : hip_fail(e);
}

}  // namespace

extern "C" {

int attn_decode_mod(const void* Q, const void* K, const void* V, void* O,
                    int B, int Hq, int Hkv, int Lk, int D,
                    float scale, const float* alibi_slopes, float softcap, int num_splits,
                    void* workspace, size_t workspace_bytes,
                    attn_dtype dtype, hipStream_t stream) {
  int S = 0;
  const int rc = decode_check(Q, K, V, O, B, Hq, Hkv, Lk, D, scale, softcap, num_splits, dtype, &S);
  if (rc != ATTN_OK) return rc;
  if (!workspace) return ATTN_ERR_NULL;
  // A workspace for one workgroup per compute unit still serves where the
  // library would choose up to two; a smaller one is refused.
  if (num_splits == 0 && workspace_bytes < attn_decode_workspace_bytes(B, Hq, D, S))
    S = std::min(S, one_round_splits(B, Hq, Hkv, Lk, compute_units()));
  const size_t need = attn_decode_workspace_bytes(B, Hq, D, S);
  if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 15)) return ATTN_ERR_WORKSPACE;
  return decode_launch(Q, K, V, O, B, Hq, Hkv, Lk, D, scale, alibi_slopes, softcap, S, workspace, dtype, stream);
}

int attn_decode_noalloc(const void* Q, const void* K, const void* V, void* O,
                        int B, int Hq, int Hkv, int Lk, int D,
                        float scale, const float* alibi_slopes, float softcap, int num_splits,
                        attn_dtype dtype, hipStream_t stream) {
  int S = 0;
  const int rc = decode_check(Q, K, V, O, B, Hq, Hkv, Lk, D, scale, softcap, num_splits, dtype, &S);
  if (rc != ATTN_OK) return rc;
  if (attn_decode_workspace_bytes(B, Hq, D, S) > attn::kDecodeScratchBytes) return ATTN_ERR_WORKSPACE;
  void* ws = nullptr;
  const hipError_t e = attn::decode_scratch(&ws);
  if (e != hipSuccess) return hip_fail(e);
  return decode_launch(Q, K, V, O, B, Hq, Hkv, Lk, D, scale, alibi_slopes, softcap, S, ws, dtype, stream);
}

int attn_decode(const void* Q, const void* K, const void* V, void* O,
                int B, int Hq, int Hkv, int Lk, int D,
                float scale, const float* alibi_slopes, int num_splits,
                void* workspace, size_t workspace_bytes,
                attn_dtype dtype, hipStream_t stream) {
  return attn_decode_mod(Q, K, V, O, B, Hq, Hkv, Lk, D, scale, alibi_slopes, 0.f, num_splits, workspace,
                         workspace_bytes, dtype, stream);
}

int attn_fwd_kernels(int D, attn_dtype dtype, int causal, int alibi, float softcap, int window,
                     char* buf, size_t len) {
  if (!std::isfinite(softcap) || softcap < 0.f || window < 0) return ATTN_ERR_SHAPE;
  if (!dims_supported(D, dtype)) return ATTN_ERR_UNSUPPORTED;
  if ((softcap > 0.f && (!causal || alibi)) || (window > 0 && !causal)) return ATTN_ERR_UNSUPPORTED;
  const attn::PrefillFlags f = attn::prefill_flags(causal != 0, alibi != 0, softcap > 0.f, window > 0);
  char s[96];
  std::snprintf(s, sizeof s, "prefill_kernel<%d,%s,%d,%d,%d,%d>", D, dtype_name(dtype), (int)f.causal, (int)f.alibi,
                (int)f.cap, (int)f.win);
  return put(buf, len, s);
}

int attn_fwd_call_kernels(int B, int Hq, int Hkv, int Lq, int Lk, int D, attn_dtype dtype, int causal, int alibi,
                          float softcap, int window, int workspace, char* buf, size_t len) {
  if (!shape_ok(B, Hq, Hkv, Lq, Lk)) return ATTN_ERR_SHAPE;
  char s[160];
  const int rc = attn_fwd_kernels(D, dtype, causal, alibi, softcap, window, s, sizeof s);
  if (rc != ATTN_OK) return rc;
  const attn::PrefillSplitPlan plan =
      attn::prefill_split_plan(B, Hq, Hkv, Lq, Lk, D, causal != 0, window, alibi != 0, softcap > 0.f, compute_units(),
                               workspace ? attn::kMaxPrefillSplits : 1);
  if (plan.kgroups > 0) {
    const int n = std::snprintf(s, sizeof s, "prefill_split_kernel<%d,%s,%d,%d,%d>", D, dtype_name(dtype), plan.kgroups,
                                alibi ? 1 : 0, softcap > 0.f ? 1 : 0);
    if (plan.splits > 1) std::snprintf(s + n, sizeof s - n, ";prefill_combine_kernel<%d,%s>", D, dtype_name(dtype));
  }
  return put(buf, len, s);
}

int attn_decode_kernels(int Hq, int Hkv, int D, attn_dtype dtype, int alibi, float softcap, char* buf, size_t len) {
  if (Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || !std::isfinite(softcap) || softcap < 0.f) return ATTN_ERR_SHAPE;
  if (!dims_supported(D, dtype)) return ATTN_ERR_UNSUPPORTED;
  const int gh = attn::decode_split_heads(Hq / Hkv);
  const int a = alibi ? 1 : 0, c = softcap > 0.f ? 1 : 0;
  char s[160];
  if (gh == 0)
    std::snprintf(s, sizeof s, "decode_mfma_kernel<%d,%s,%d,%d>;decode_combine_kernel<%d,%s>", D, dtype_name(dtype), a,
                  c, D, dtype_name(dtype));
  else
    std::snprintf(s, sizeof s, "decode_split_kernel<%d,%s,%d,%d,%d>;decode_combine_kernel<%d,%s>", D,
                  dtype_name(dtype), gh, a, c, D, dtype_name(dtype));
  return put(buf, len, s);
}

int peaks_hbm_read(const void* buf, size_t bytes, float* sink, hipStream_t stream) {
  if (!buf || !sink || bytes < 16 || bytes % 16 || (reinterpret_cast<uintptr_t>(buf) & 15)) return ATTN_ERR_SHAPE;
  const hipError_t e = attn::launch_hbm_read(buf, bytes, sink, stream);
  return e == hipSuccess ? ATTN_OK : hip_fail(e);
}

int peaks_hbm_read_sink_floats(void) { return attn::hbm_read_sink_floats(); }

int peaks_mfma(int dtype, int iters, const void* operands, float* sink, unsigned long long* clocks,
               hipStream_t stream) {
  if (!operands || !sink || !clocks || iters < 1 || (dtype != 0 && dtype != 1)) return ATTN_ERR_SHAPE;
  const hipError_t e = attn::launch_mfma_loop(dtype, iters, operands, sink, clocks, stream);
  return e == hipSuccess ? ATTN_OK : hip_fail(e);
}

int peaks_mfma_waves(void) { return attn::mfma_loop_waves(); }

size_t peaks_mfma_operand_bytes(void) { return attn::mfma_loop_operand_bytes(); }

int norm_chunks(int rms, int N, int M, norm_dtype dtype) {
  if (N < 1 || M < 1 || (dtype != NORM_F16 && dtype != NORM_BF16 && dtype != NORM_F32)) return 0;
  // One chunk per row means one kernel (a wave or a workgroup per row), X
  // read once.  It pays when
  //  - a row has at most 64 KiB: a row's time in one workgroup is then below
  //    that of a second kernel (64 x 32768 bf16 RMSNorm 4.1 us, 5.9 with 8
  //    chunks; L2 64 x 16384 fp32 3.9 against 5.1; at 128 KiB 7.8 against
  //    6.7 for 64 rows);
  //  - half the compute units have a row of at most 208 KiB: there the L2 norm
  //    has its line (128 fp32 rows: 208 KiB 9.2 us against 9.4 with 4 chunks,
  //    240 KiB 10.4 against 9.8; bf16 160 KiB 7.9 and 8.7, 208 KiB 9.9 and 9.6),
  //    while RMSNorm gains up to what it holds (128 rows of 256 KiB 14.5 against
  //    15.7, 200 18.4 against 28.9), which the next line takes only with more
  //    rows;
  //  - the rows fill at least 85 % of the compute units' rounds and, for
  //    RMSNorm, a row fits the workgroup's registers (256 x 2^17: RMSNorm
  //    1.19x the two kernels with 2 chunks, the L2 norm 1.03x; but L2 300 x
  //    2^17 fp32 31 us against 29 with 2 chunks).
  const int64_t elem = dtype == NORM_F32 ? 4 : 2, cu = compute_units(), row = M * elem;
  const int64_t rounds = (N + cu - 1) / cu;
  if (attn::norm_one_kernel(rms != 0, M, (int)elem, 1) &&
      (row <= 65536 || (2 * (int64_t)N >= cu && row <= 212992) || (N >= cu && (int64_t)N * 100 >= rounds * cu * 85)))
    return 1;
  // Otherwise about two workgroups per compute unit (measured on the 256 x
  // 2^17 row reductions: 2 chunks per row beat 4, 8 and 16), chunks of at
  // least 4096 elements.
  constexpr int kTargetBlocks = 512, kMinChunk = 4096;
  int64_t c = (kTargetBlocks + N - 1) / N;
  const int64_t cmax = ((int64_t)M + kMinChunk - 1) / kMinChunk;
  if (c > cmax) c = cmax;
  return c < 1 ? 1 : (int)c;
}

int norm_kernels(int rms, int M, norm_dtype dtype, int chunks, char* buf, size_t len) {
  if (dtype != NORM_F16 && dtype != NORM_BF16 && dtype != NORM_F32) return ATTN_ERR_UNSUPPORTED;
  const int elem = dtype == NORM_F32 ? 4 : 2;
  if (M < 1 || M % (16 / elem) || chunks < 1) return ATTN_ERR_SHAPE;
  const char* t = dtype == NORM_F32 ? "f32" : dtype == NORM_BF16 ? "bf16" : "f16";
  char s[96];
  if (attn::norm_one_kernel(rms != 0, M, elem, chunks))
    std::snprintf(s, sizeof s, "%s_row_kernel<%s>", rms ? "rms" : "l2", t);
  else if (rms)
    std::snprintf(s, sizeof s, "norm_split_kernel<%s,1>;rms_apply_kernel<%s>", t, t);
  else
    std::snprintf(s, sizeof s, "norm_split_kernel<%s,0>;l2_combine_kernel", t);
  return put(buf, len, s);
}

size_t norm_workspace_bytes(int N, int chunks) {
  if (N < 1 || chunks < 1) return 0;
  const size_t bytes = (size_t)N * chunks * 2 * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}

}  // extern "C"

namespace {

int norm_run(const void* X, void* Y, float* out, int N, int M, float eps, norm_dtype dtype, int chunks,
             void* workspace, size_t workspace_bytes, bool rms, hipStream_t stream) {
  if (!X || !out || !workspace || (rms && !Y)) return ATTN_ERR_NULL;
  if (dtype != NORM_F16 && dtype != NORM_BF16 && dtype != NORM_F32) return ATTN_ERR_UNSUPPORTED;
  const int vec = dtype == NORM_F32 ? 4 : 8;
  if (N < 1 || M < 1 || M % vec || chunks < 0 || !std::isfinite(eps) || eps < 0.f) return ATTN_ERR_SHAPE;
  if ((int64_t)N * M >= (int64_t(1) << 40)) return ATTN_ERR_SHAPE;
  const int C = chunks ? chunks : norm_chunks(rms ? 1 : 0, N, M, dtype);
  if ((int64_t)N * C > kMaxGrid) return ATTN_ERR_SHAPE;
  if (workspace_bytes < norm_workspace_bytes(N, C) || (reinterpret_cast<uintptr_t>(workspace) & 15))
    return ATTN_ERR_WORKSPACE;
  attn::NormParams p{};
  p.x = X; p.y = Y; p.out = out;
  p.ws_r = static_cast<float*>(workspace);
  p.ws_t = p.ws_r + (size_t)N * C;
  p.N = N; p.M = M; p.chunks = C;
  const int64_t per = ((int64_t)M + C - 1) / C;
  p.chunk = (int)((per + vec - 1) / vec * vec);
  p.dtype = (int)dtype;
  p.rms = rms ? 1 : 0;
  p.eps = eps;
  p.invM = 1.f / (float)M;
  const hipError_t e = attn::launch_norm(p, stream);
  return e == hipSuccess ? ATTN_OK : hip_fail(e);
}

}  // namespace

extern "C" {

int norm_l2(const void* X, float* out, int N, int M, norm_dtype dtype, int chunks,
            void* workspace, size_t workspace_bytes, hipStream_t stream) {
  return norm_run(X, nullptr, out, N, M, 0.f, dtype, chunks, workspace, workspace_bytes, false, stream);
}

int rmsnorm_rowmax(const void* X, void* Y, float* rowmax, int N, int M, float eps, norm_dtype dtype,
                   int chunks, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  return norm_run(X, Y, rowmax, N, M, eps, dtype, chunks, workspace, workspace_bytes, true, stream);
}

}  // extern "C"
