// Shared declarations of libpvf's translation units (host side + small device helpers).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pvf.h"

namespace pvf {

typedef __bf16 bf16_t;

// ---- error reporting ---------------------------------------------------------------
// Records a printf-style message on the context (or in a thread-local slot if ctx == NULL).
void set_error(pvf_ctx *ctx, const char *fmt, ...);

#define PVF_HIP_CHECK(ctx, call)                                                         \
  do {                                                                                   \
    hipError_t e__ = (call);                                                             \
    if (e__ != hipSuccess) {                                                             \
      ::pvf::set_error(ctx, "%s: %s (%s:%d)", #call, hipGetErrorString(e__), __FILE__,  \
                       __LINE__);                                                        \
      return PVF_EHIP;                                                                   \
    }                                                                                    \
  } while (0)

#define PVF_LAUNCH_CHECK(ctx, what) PVF_HIP_CHECK(ctx, hipGetLastError())

#define PVF_REQUIRE(ctx, cond, code, ...)                                                \
  do {                                                                                   \
    if (!(cond)) {                                                                       \
      ::pvf::set_error(ctx, __VA_ARGS__);                                                \
      return code;                                                                       \
    }                                                                                    \
  } while (0)

// ---- device helpers ------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}
__device__ __forceinline__ float to_float(float x) { return x; }
__device__ __forceinline__ float to_float(bf16_t x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_float(float x);
template <> __device__ __forceinline__ float from_float<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_float<bf16_t>(float x) { return (bf16_t)x; }

constexpr int kWave = 64;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}

// ---- kernel launchers (each defined in the .hip file holding its kernels) -------------
// Row filter of the epilogue's stage 1: which logits rows exist and where their summary goes.
struct RowFilter {
  const int32_t *n_drafts;  // [G] or NULL (NULL: every row is live, out row = in row)
  const int32_t *done;      // [G]
  const int32_t *k_active;  // [G]
  const int32_t *seq_slot;  // [n_seq] compact sequence -> slot g*(1+K)+j (negative: no sequence), or NULL (identity)
  int32_t slots_per_group;  // 1+K
  int32_t R, prompt_len, block_len, T;
};

// Where a logits row's summary goes (-1: nowhere) and whether the row exists at all.
__device__ __forceinline__ bool row_target(const RowFilter &rf, int64_t row, int64_t *out_row) {
  *out_row = row;
  if (rf.n_drafts == nullptr) return true;
  const int s = (int)(row / rf.R), r = (int)(row % rf.R);
  const int slot = rf.seq_slot ? rf.seq_slot[s] : s;
  if (slot < 0) { *out_row = -1; return false; }
  const int g = slot / rf.slots_per_group, j = slot % rf.slots_per_group;
  *out_row = (int64_t)slot * rf.R + r;
  if (rf.done[g] || j > rf.n_drafts[g]) return false;
  return rf.prompt_len + rf.k_active[g] * rf.block_len + r < rf.T;
}

// Keys per row of a key-contiguous value buffer: T rounded up to a whole tile of the attention kernel.
inline int vt_keys(int T) { return (T + 63) / 64 * 64; }

pvf_status launch_stage1(pvf_ctx *ctx, hipStream_t s, const void *logits, int dtype,
                         int64_t n_rows, int vocab, int mask_id, float scale,
                         const RowFilter &rf, float *conf, int32_t *tok, float *ent = nullptr);

// rows of the decision window: min(c * block_len, gen_len), c = 2, or 4 with n_sparse > 0
int window_rows(const pvf_decode_cfg &c);

// entropy of short logits rows (calibration only); rows are filtered like stage 1.  launch_stage1 with ent != NULL takes rows
// of any length (conf and tok may then be NULL).
pvf_status launch_entropy_short(pvf_ctx *ctx, hipStream_t s, const void *logits, int dtype,
                          int64_t n_rows, int vocab, int mask_id, float scale,
                          const RowFilter &rf, float *ent);

pvf_status launch_plan_vocab_select(pvf_ctx *ctx, hipStream_t s, const uint32_t *cal_n,
                                    const uint32_t *cal_m, const uint32_t *cal_a,
                                    const double *cal_vig, int vocab, int mask_id, uint32_t n_min,
                                    uint32_t m_min, float rho_ver, float gamma_vig,
                                    uint32_t *plan_bitmap);

// status (NULL: none; may be pinned host memory): status[5 g ..] = done, n_drafts, n_commit[0..2] of group g after the round.
// skip_if_zero (NULL: never): device word; where it holds 0 the state stays as it is.
struct Stage2Out {
  int32_t *status = nullptr;
  const int32_t *skip_if_zero = nullptr;
};
pvf_status launch_stage2(pvf_ctx *ctx, hipStream_t s, int G, int vocab, int mask_id,
                         const uint32_t *plan_bitmap, const pvf_decode_cfg &cfg,
                         const pvf_state &st, const Stage2Out &out = Stage2Out{});

pvf_status launch_state_init(pvf_ctx *ctx, hipStream_t s, const int32_t *prompt, int G,
                             int mask_id, const pvf_decode_cfg &cfg, const pvf_state &st);

// builds seq_slot[] and row_pos[] for a round; n_seq entries are written (padding repeats the first live canvas, slot 0 where
// none is)
pvf_status launch_build_batch(pvf_ctx *ctx, hipStream_t s, int G, int n_seq,
                              const pvf_decode_cfg &cfg, const pvf_state &st,
                              int32_t *seq_slot, int32_t *row_pos);

// the same, n_seq being an upper bound: *n_live = number of live slots, at most n_seq (pad: slot 0 where none is); entries behind
// them are -1, without window rows; and the embedding of their canvases (float32), h[s * T + t]
pvf_status launch_embed_batch(pvf_ctx *ctx, hipStream_t s, int G, int n_seq, const pvf_decode_cfg &cfg, const pvf_state &st,
                              const float *embed, int d, int vocab, bool pad, int32_t *seq_slot, int32_t *row_pos, int32_t *n_live, float *h);

// block-level K/V cache (kvcache.hip)
pvf_status launch_fill_row_pos(pvf_ctx *ctx, hipStream_t s, const pvf_decode_cfg &cfg, const pvf_state &st,
                               const int32_t *seq_slot, int n_seq, int32_t *row_pos);
pvf_status launch_kv_store(pvf_ctx *ctx, hipStream_t s, int dtype, const void *qkv, const void *vt,
                           const int32_t *seq_slot, int slots_per_group, int S, int T, int d,
                           void *kc, void *vc, void *vtc, int64_t group_stride);   // vt, vtc: rows of vt_keys(T) keys
pvf_status launch_embed_rows(pvf_ctx *ctx, hipStream_t s, int dtype, const void *embed, const int32_t *canvas,
                             const int32_t *seq_slot, const int32_t *row_pos, int n_rows, int R, int T,
                             int d, int vocab, void *out);
pvf_status launch_rope_rows(pvf_ctx *ctx, hipStream_t s, int dtype, void *qkv, const int32_t *row_pos,
                            int n_rows, int T, int n_heads, int d_head, const float2 *cos_sin);
pvf_status launch_attention_window(pvf_ctx *ctx, hipStream_t s, int dtype, const void *qkv_w, const void *kc,
                                   const void *vc, int64_t group_stride, const pvf_decode_cfg &cfg,
                                   const pvf_state &st, const int32_t *seq_slot, int n_seq, int n_heads,
                                   int d_head, void *out);

pvf_status launch_copy_out(pvf_ctx *ctx, hipStream_t s, int G, int K, int T,
                           const int32_t *canvas, int32_t *out_tokens);

// forward building blocks
// ss (bf16 only, may be NULL): ss[m] = sum of squares of row m
pvf_status launch_embed(pvf_ctx *ctx, hipStream_t s, int dtype, const void *embed,
                        const int32_t *tokens, const int32_t *seq_slot, int S, int T, int d,
                        int vocab, void *h, float *ss = nullptr);
// out[n, k] = bf16(w[n, k] * gain[k])
pvf_status launch_fold_gain(pvf_ctx *ctx, hipStream_t s, const void *w, const void *gain, void *out, int64_t n, int k);
pvf_status launch_rmsnorm(pvf_ctx *ctx, hipStream_t s, int dtype, const void *x,
                          const void *gain, void *out, int M, int d, float eps);
pvf_status launch_gather_rows(pvf_ctx *ctx, hipStream_t s, int dtype, const void *h,
                              const int32_t *row_pos, int S, int T, int R, int d, void *out);
pvf_status launch_rope(pvf_ctx *ctx, hipStream_t s, int dtype, void *qkv, int M, int T,
                       int n_heads, int d_head, const float2 *cos_sin);
enum GemmEpilogue { kEpiStore = 0, kEpiResidual = 1, kEpiSwiglu = 2, kEpiQkvRope = 3, kEpiPartial = 4, kEpiQkvWindow = 5, kEpiQkvRopeWin = 6 };
// RMSNorm folded into the projections around it (bf16 MFMA GEMMs of launches above the split-K range):
// the projection that writes the residual stream also writes, per `slot` of 256 (or 64) columns, the sum of
// squares of each row's (rounded) values, ss[slot * ld + m]; the projection that reads the stream takes h
// itself as its operand, with the gain folded into its weights, and multiplies row m of its accumulators by
// rsqrt(sum over slots of ss / d + eps) in its epilogue.
struct NormArgs {
  float *ss_out = nullptr;        // kEpiResidual: where the row sums of squares of this launch go
  const float *ss_in = nullptr;   // kEpiSwiglu / kEpiQkvRope: row sums of squares of the operand rows
  int32_t n_slots_in = 0, ld = 0; // slots to add up; rows per slot
  int32_t group_in = 1;           // 4: slots of 64 columns, four are added up first
  float inv_d = 0.f, eps = 0.f;
};
// Rotary embedding of one pair: a = element i of a head, b = element i + d_head / 2 -> (a cos - b sin, b cos + a sin).  Written
// out as one rounded product and one fused multiply-add each, so that every kernel that rotates bf16 rows of 128-wide heads (the
// QKV projection's epilogue, the passes of their own) gives the same bits: which of them a launch takes depends on its size,
// and left to itself the compiler contracted the sum differently from place to place (6e-6 of the elements differed).
__device__ __forceinline__ float2 rotate_pair(float a, float b, float cos, float sin) {
#pragma clang fp contract(off)
  return make_float2(__builtin_fmaf(a, cos, -(b * sin)), __builtin_fmaf(a, sin, b * cos));
}
// Rotary embedding in the epilogue of a float32 QKV projection: row m is canvas position m % T, or row_pos[m] (negative:
// a padding row, rotated like position T - 1); cos_sin [T][half].
struct RopeF32 {
  const float2 *cos_sin;
  const int32_t *row_pos;         // NULL: whole canvases
  int32_t T, half;
};
// Rows of a float32 projection.
struct RowsF32 {
  const float *gain = nullptr;    // the operand is RMSNorm(A) * gain
  float eps = 0.f;
  double inv_k = 0.0;             // 1 / row length
  const int32_t *map = nullptr;   // row s * R + r is row s * T + map[s * R + r] of A and of the residual (zeros outside [0, T))
  int32_t T = 0, R = 0;
  const int32_t *n_live = nullptr;   // device: only the first *n_live * per_seq rows are computed
  int32_t per_seq = 0;
};
// out = RMSNorm(x) * gain by rows.gain, eps, inv_k (and n_live); the norm of every float32 row of up to kNormF32Max elements
constexpr int kNormF32Max = 1024;
pvf_status launch_rmsnorm_f32(pvf_ctx *ctx, hipStream_t s, const float *x, float *out, int M, int K, const RowsF32 &rows);
// C[M,N] = A[M,K] W[N,K]^T; kEpiResidual adds residual[M,N]; kEpiSwiglu: W is [2N,K] (gate|up),
// C[M,N] = silu(gate) * up.
pvf_status launch_gemm(pvf_ctx *ctx, hipStream_t s, int dtype, GemmEpilogue epi, const void *A,
                       const void *W, void *C, const void *residual, int M, int N, int K, bool split_ok = true);
// Pieces of the split-K path for launches of few rows.
// out[M, N] = epilogue(sum over splits of partial[z][M][Nw]) in split order (store, + residual, SwiGLU of gate | up halves)
pvf_status launch_splitk_finalize(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const float *partial, int splits,
                                  int M, int N, void *C, const void *residual);
// h[m, :] <- h[m, :] + sum over splits of partial[z][m][:] (rounded once), then out[m, :] = RMSNorm(h[m, :]) * gain
pvf_status launch_reduce_residual_rmsnorm(pvf_ctx *ctx, hipStream_t s, const float *partial, int splits, int M, int d,
                                          void *h, const void *gain, void *out, float eps);
bool reduce_residual_rmsnorm_supported(int dtype, int d);

pvf_status launch_fill_normal(pvf_ctx *ctx, hipStream_t s, int dtype, void *dst, int64_t n,
                              uint64_t seed, float mean, float std);

}  // namespace pvf
