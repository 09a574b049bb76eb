// Internal declarations shared by the translation units of libcitrus.so.
// Not part of the public ABI (see include/citrus.h for that).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "citrus.h"

namespace citrus {

// A strided [B, L, H, S, d] view in element units; d is contiguous.
struct View {
  const void* ptr;
  int64_t sb, sl, sh, ss;
};

inline View make_view(const citrus_tensor& t) { return View{t.ptr, t.stride_b, t.stride_l, t.stride_h, t.stride_s}; }

// Problem sizes every kernel launcher receives.
struct Dims {
  int B, L, Hq, Hkv, G, D;
  float scale;  // softmax scale (already resolved, never 0)
};

// The candidate keys/values of a step: cache rows then chunk rows.
struct Segments {
  View cache;   // [B, L, Hkv, >= n_c, d]
  View chunk;   // [B, L, Hkv, c, d]
  int n_c;      // valid cache rows
  int c;        // chunk rows
};

// Scores of B*L*Hkv units: candidate j of unit u has the sum over x < sums, in this order, of ptr[(u * sums + x) * n + j].
struct ScoreSums {
  const float* ptr;
  int sums;
};

// The eviction of one cache, a selection per KV head: of the first n candidates of [cache ; chunk] the k best stay, in
// order, followed by the last `appended` candidates.
struct Eviction {
  Segments ks, vs;
  ScoreSums score;  // not read while n <= k, unless acc_new is given: the kept states then take their sums along
  int n, k, forced, appended;
  int32_t* idx;     // optional, pitch k
  View k_new, v_new;
  const float* acc;  // optional: sums that the cache's states carry (added to their scores) ...
  float* acc_new;    // ... and that the kept states take along; [B*L*Hkv][acc_pitch]
  int acc_pitch;
};
// Every candidate stays, and no scores are carried on: none are formed.
inline bool gather_only(const Eviction& e) { return e.n <= e.k && e.acc_new == nullptr; }
inline citrus_status hip_status(hipError_t e) { return e == hipSuccess ? CITRUS_OK : CITRUS_ERR_DEVICE; }

// ---- kernels of the f32 mode, attn_generic.hip ----
// rows: number of query rows per head; causal != 0 -> row t sees candidates j <= n_c + t.
// out may be NULL (log-sum-exp only); lse may be NULL.
hipError_t launch_attn_f32(const Dims& dm, View q, int rows, Segments kseg, Segments vseg, int causal, View out,
                           float* lse, hipStream_t st);
// score[b,l,g,j] = sum_{h in g} sum_{t<rows} exp(scale*q.k - lse[b,l,h,t]) (0 where masked)
hipError_t launch_colsum_f32(const Dims& dm, View q, int rows, Segments kseg, int causal, const float* lse,
                             float* score, hipStream_t st);

// score[b,l,g,j] = sum_{h in g} sum_{t<rows} softmax_j(scale*q.k); lse_scratch: B*L*Hq*rows floats
hipError_t launch_instr_score_f32(const Dims& dm, View q, int rows, Segments kseg, float* lse_scratch, float* score,
                                  hipStream_t st);
// The causal attention of kseg.c rows and the instruction score in one launch, with the bits of the two.  evict (optional): the
// eviction by these scores as well.
bool attn_score_f32_in_one_launch(const Dims& dm, int rows, int instr_rows, int n);
// May, and should, the launch evict by its scores as well?
bool step_f32_in_one_launch(const Dims& dm, const Eviction& evict);
hipError_t launch_attn_score_f32(const Dims& dm, View q, Segments kseg, Segments vseg, View out, View q_instr, int instr_rows,
                                 float* score, const Eviction* evict, hipStream_t st);

// ---- bf16 MFMA kernels (head_dim 64 and 128: every bf16 configuration), attn_mfma.hip ----
bool mfma_path_supported(int dtype, const Dims& dm);
// The chunk's kseg.c query rows over [cache ; chunk], row t over candidates j <= n_c + t.
// lse (optional): the rows' log-sum-exp (natural log).  lse_cache (optional, kseg.n_c > 0): the same over the cache
// states alone, a by-product.
// q_rope_pos0 >= 0: the query rows are given without rotary embedding and are
// rotated to positions q_rope_pos0 + row inside the kernel, with the bits launch_rope would give.
hipError_t launch_attn_mfma(const Dims& dm, View q, Segments kseg, Segments vseg, View out, float* lse, float* lse_cache,
                            hipStream_t st, int q_rope_pos0 = -1, float rope_base = 0.f);
// Column sums, colsum.hip.  norm[row * norm_pitch]: the rows' normalisers; times to_log2 they are in the log2 domain.
hipError_t launch_colsum_mfma(const Dims& dm, View q, int rows, Segments kseg, int causal, const float* norm, int norm_pitch,
                              float to_log2, float* score, hipStream_t st);
// Most ranges of key tiles a two-launch score splits the keys of a row into (one workgroup per range).
constexpr int kMaxKeySplits = 8;
// Floats of scratch that cover every launch_instr_score_mfma call with at most `rows` query rows per head over
// at most n keys (the launcher picks its kernel by the call's own shape, and the kernels' needs do not grow
// together: a block sized for the largest shape alone could be too small for a smaller one).
size_t instr_score_mfma_workspace_floats(const Dims& dm, int rows, int n);
// `workspace_floats`: what the block behind `workspace` holds; the kernel is chosen by the call's shape alone, and
// hipErrorInvalidValue comes back if its scratch does not fit.
// sums (optional): what it points to is {score, 1}; a kernel that forms partial sums per key may leave them in the
// workspace and describe them there instead of adding them up to `score`.
hipError_t launch_instr_score_mfma(const Dims& dm, View q, int rows, Segments kseg, float* workspace,
                                   size_t workspace_floats, float* score, hipStream_t st, ScoreSums* sums = nullptr);

// compute units of the current device, looked up once per device (instr_strip.hip)
int compute_units();

// ---- instruction score with one q.k product per (row, key): row strips kept on chip, instr_strip.hip ----
// taken for this shape?
bool instr_strip_supported(const Dims& dm, const View& q, int rows, const Segments& kseg);
int instr_strip_rows(const Dims& dm, int rows, int n);  // of a strip: 32 or 64
// largest scratch any supported launch with at most `rows` rows and at most n keys writes (0: none is supported)
size_t instr_strip_workspace_floats(const Dims& dm, int rows, int n);
hipError_t launch_instr_strip(const Dims& dm, View q, int rows, Segments kseg, float* workspace, size_t workspace_floats,
                              float* score, hipStream_t st, ScoreSums* sums = nullptr);

// What a strip kernel's partial columns still need: nothing for one strip (its column is `score`), a description for a
// caller who adds them, else a launch that does.
hipError_t finish_strip_scores(const Dims& dm, const float* part, int strips, int n, float* score, hipStream_t st,
                               ScoreSums* sums);

// ---- chunk attention and instruction score of a small step in one launch, attn_mfma.hip ----
// The same bits as the two launches.  Both read [cache ; chunk]; q_instr: instr_rows rows per head.
bool attn_score_in_one_launch(const Dims& dm, const Segments& kseg, const Segments& vseg, const View& q_instr, int instr_rows);
// evict (optional): the eviction by these scores, made by the launch (tickets: B*L*Hkv of them, zero; zero again afterwards).
// Otherwise sums as in launch_instr_score_mfma.  hipErrorInvalidValue if the strips' columns do not fit workspace_floats.
hipError_t launch_attn_score_mfma(const Dims& dm, View q, Segments kseg, Segments vseg, View out, int q_rope_pos0,
                                  float rope_base, View q_instr, int instr_rows, float* workspace, size_t workspace_floats,
                                  float* score, hipStream_t st, ScoreSums* sums, const Eviction* evict, int32_t* tickets);
// Does that launch need its tickets?  (n: the step's candidates)
bool step_needs_tickets(const Dims& dm, int instr_rows, int n, const Eviction& evict);
hipError_t launch_clear_tickets(const Dims& dm, int32_t* tickets, hipStream_t st);

// ---- bf16 MFMA decoding step (at most 32 query heads per KV head), decode_attn.hip ----
bool decode_mfma_supported(int dtype, const Dims& dm);
size_t decode_mfma_workspace_floats(const Dims& dm);
// One query row per head over [cache ; the new token's row] (kseg.c == 1); workspace holds the partial
// results of the key ranges (decode_mfma_workspace_floats).  append_token != 0: the token's K/V row is
// also written to row kseg.n_c of the cache tensors (which must have room for it).
hipError_t launch_decode_mfma(const Dims& dm, View q, Segments kseg, Segments vseg, View out, float* workspace,
                              int append_token, hipStream_t st);

// ---- rotary embedding at explicit positions, rope.hip ----
// y[b,l,h,s,:] = RoPE(x[b,l,h,s,:], pos0 + s) for h < heads, s < rows; y may be x itself.
hipError_t launch_rope(int dtype, const Dims& dm, View x, View y, int heads, int rows, int pos0, float base,
                       hipStream_t st);
// Up to kMaxRopeJobs rotations in one launch (bf16; f32 takes one launch each): the keys and queries of a step.
// A job with rows <= 0 is skipped.
constexpr int kMaxRopeJobs = 4;
struct RopeJob {
  View x, y;
  int heads, rows, pos0;
};
hipError_t launch_rope_batch(int dtype, const Dims& dm, const RopeJob* jobs, int count, float base, hipStream_t st);

// Kernels that take more than 64 KB of dynamic LDS need their limit raised once per device.  `state` is a
// static object next to the launch; the current device's slot remembers the largest size granted.  The
// slots are atomics (relaxed order is enough: the value only saves a repeated hipFuncSetAttribute, which
// the runtime serialises itself), so host threads may call the launchers concurrently.  Every launcher
// asks for ONE size per kernel (its maximum), so two threads can never lower each other's limit.
constexpr int kMaxDevices = 64;
struct LdsLimit {
  std::atomic<int> granted[kMaxDevices] = {};
};
inline hipError_t raise_lds_limit(LdsLimit& state, const void* kernel, int bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < kMaxDevices;
  if (tracked && state.granted[dev].load(std::memory_order_relaxed) >= bytes) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && tracked) {
    int seen = state.granted[dev].load(std::memory_order_relaxed);
    while (seen < bytes && !state.granted[dev].compare_exchange_weak(seen, bytes, std::memory_order_relaxed)) {
    }
  }
  return e;
}

// ---- selection and compaction, select_compact.hip ----
// units = B*L*Hsel; score rows are [units*(per_layer?Hkv:1)] x n.
hipError_t launch_topk(const float* score, int units, int heads_to_sum, int n, int k, int forced, int32_t* idx,
                       hipStream_t st);
// score [B*L*Hkv][n] += acc [B*L*Hkv][acc_pitch] on the first n_c candidates
hipError_t launch_score_add(const Dims& dm, float* score, const float* acc, int n, int n_c, int acc_pitch,
                            hipStream_t st);
// acc_new [B*L*Hkv][acc_pitch]: row r < m takes score[idx[r]] (idx as in launch_compact)
hipError_t launch_score_gather(const Dims& dm, const float* score, const int32_t* idx, float* acc_new, int n, int m,
                               int idx_pitch, int idx_heads, int acc_pitch, hipStream_t st);
// Output rows 0 .. kept - 1: the candidates idx names; behind them the last `appended` candidates in order.
// acc_new (optional) [B*L*Hkv][acc_pitch]: row r < kept also takes score[idx[r]] of score [B*L*Hkv][n].
hipError_t launch_compact(int elem_bytes, const Dims& dm, Segments kseg, Segments vseg, const int32_t* idx,
                          int idx_pitch, int idx_heads, int kept, int appended, View k_new, View v_new,
                          const float* score, int n, float* acc_new, int acc_pitch, hipStream_t st);

// May, and should, the eviction of a cache that keeps `rows` rows per head, ranking n candidates, be one launch?
bool evict_in_one_launch(int elem_bytes, const Dims& dm, int n, int rows);
// One or two evictions in one launch.
hipError_t launch_evict(int elem_bytes, const Dims& dm, const Eviction* e, int count, hipStream_t st);

}  // namespace citrus
