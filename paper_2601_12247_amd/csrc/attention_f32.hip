// float32 attention with float64 sums on the matrix cores (the float32 path of the forward): out = softmax(q k^T /
// sqrt(d_head)) v over all T keys of a canvas, no mask of any kind (the denoiser sees the whole canvas, Sec. 2).
// Full canvases, or the window rows of a K/V-cached round, whose keys come from the window itself or from the
// cache of the canvas' group.  d_head a multiple of 16, any T whose scores fit into LDS.
//
// One workgroup = 16 queries of one (canvas, head), four waves.  Bound by the SIMDs' issue (a v_mfma_f64_16x16x4_f64 takes 64
// cycles, in which its SIMD issues no vector instruction of any wave) and, in the small parity model, by latency:
//   * scores: the waves take every fourth tile of 16 keys; operands come from global memory in operand layout
//     (16 bytes per lane = four consecutive d, the contraction permuted alike in q and k), the next tile's while
//     this one's are multiplied; scores are rounded to float32 into LDS, rows padded against bank conflicts;
//   * softmax in float32 like the plain kernel: four rows per wave side by side; weights are divided by their row's sum before
//     the four waves read them, each of which would divide all of them again;
//   * out: the waves take every fourth 16 columns of the head, all keys, so that nothing is added across waves;
//     two accumulators alternate because a float64 MFMA that waits for the previous one idles the pipe; values are
//     fetched four tiles ahead, the first ones before the softmax (a tile is 256 cycles of MFMA, a load 1500);
//   * loads of whole canvases are a lane offset that stays and a descriptor whose base moves by scalar arithmetic: with 64-bit
//     addresses a tile of values (4 MFMAs) took 57 vector instructions, 300 cycles beside the MFMAs' 256, now 17.
// Measured (per layer; plain kernel, 64-bit addresses, now): 1-3 canvases x 128 tokens 28, 8.8, 8.5 us; 20 canvases x 229 tokens 39 ->
// 36, 40 x 229 72 -> 65; 4 x 512 with 8 heads of 128 121 -> 107.
#include "common.h"

namespace pvf {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int TQ = 16;

struct WinF32 {
  const float *kc, *vc;                // cache rows [T][d] of this layer, group 0
  int64_t group_stride;
  const int32_t *seq_slot, *k_active;
  int32_t slots_per_group, prompt_len, block_len;
};

#ifdef __HIP_DEVICE_COMPILE__          // the descriptor type does not exist in the host pass
// Descriptor of what begins at x; every offset used with it lies inside the caller's canvas.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_from(const float *x) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, -16, 0x00020000);
}
#endif

template <int KC, bool WIN>            // KC = d_head / 16
__global__ void __launch_bounds__(256)
attention_f32_kernel(const float *__restrict__ qkv, float *__restrict__ out, int n_rows, int T, int n_heads,
                     float inv_sqrt_dh, const int32_t *__restrict__ n_live, WinF32 wa) {
  constexpr int dh = KC * 16;
  extern __shared__ float s_p[];       // [TQ][T16 + 4]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fq = lane >> 4;
  const int q0 = blockIdx.x * TQ, head = blockIdx.y, seq = blockIdx.z;
  const int d = n_heads * dh;
  const int64_t ld = 3 * (int64_t)d;
  const int live = n_live ? *n_live : 0;              // asked for beside the first loads, not in front of them
  const float *fresh = qkv + (int64_t)seq * n_rows * ld + (int64_t)head * dh;      // q; k at + d, v at + 2 d
  const int n_tiles = (T + 15) / 16, stride = n_tiles * 16 + 4;
  int w0 = 0, w1 = T;                  // keys [w0, w1) are rows of this launch
  const float *kcb = nullptr, *vcb = nullptr;
  if (WIN) {
    const int g = wa.seq_slot[seq] / wa.slots_per_group;
    w0 = wa.prompt_len + wa.k_active[g] * wa.block_len;
    w1 = w0 + min(n_rows, T - w0);
    kcb = wa.kc + g * wa.group_stride + (int64_t)head * dh;
    vcb = wa.vc + g * wa.group_stride + (int64_t)head * dh;
  }
  auto k_row = [&](int key) -> const float * {
    key = min(key, T - 1);
    return (!WIN || (key >= w0 && key < w1)) ? fresh + d + (int64_t)(key - w0) * ld : kcb + (int64_t)key * d;
  };
  auto v_row = [&](int key) -> const float * {
    key = min(key, T - 1);
    return (!WIN || (key >= w0 && key < w1)) ? fresh + 2 * d + (int64_t)(key - w0) * ld : vcb + (int64_t)key * d;
  };

  // Whole canvases: keys and values through descriptors whose base is the tile's first row (scalar arithmetic), so that a load
  // costs no vector instruction; the last tile's rows past the end are the canvas' last one.
  const uint32_t ld4 = (uint32_t)ld * 4u;
  const int last_rows = T - (n_tiles - 1) * 16;                     // 1..16
  const uint32_t k_off = fr * ld4 + 16u * fq, k_last = min(fr, last_rows - 1) * ld4 + 16u * fq;
  uint32_t v_off[4], v_last[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v_off[e] = (4 * fq + e) * ld4 + 4u * fr, v_last[e] = min(4 * fq + e, last_rows - 1) * ld4 + 4u * fr;

  // ---- scores ----
  float4 q[KC];
  {
    const float *qr = fresh + (int64_t)min(q0 + fr, n_rows - 1) * ld;
#pragma unroll
    for (int c = 0; c < KC; ++c) q[c] = *reinterpret_cast<const float4 *>(qr + c * 16 + 4 * fq);
  }
  float4 kb[2][KC];
  auto fetch_k = [&](int buf, int kt) {
    if constexpr (!WIN) {
#ifdef __HIP_DEVICE_COMPILE__
      const auto rs = rows_from(fresh + d + (int64_t)kt * 16 * ld);
      const uint32_t o = kt == n_tiles - 1 ? k_last : k_off;
#pragma unroll
      for (int c = 0; c < KC; ++c) kb[buf][c] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, o + 64 * c, 0, 0));
#endif
      return;
    }
    const float *kr = k_row(kt * 16 + fr);
#pragma unroll
    for (int c = 0; c < KC; ++c) kb[buf][c] = *reinterpret_cast<const float4 *>(kr + c * 16 + 4 * fq);
  };
  auto score = [&](int buf, int kt) {
    doublex4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = s0;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      s0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)q[c].x, (double)kb[buf][c].x, s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)q[c].y, (double)kb[buf][c].y, s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)q[c].z, (double)kb[buf][c].z, s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)q[c].w, (double)kb[buf][c].w, s1, 0, 0, 0);
    }
    const int key = kt * 16 + fr;
#pragma unroll
    for (int e = 0; e < 4; ++e)        // row 4 e + lane / 16 = query, column lane % 16 = key
      s_p[(4 * e + fq) * stride + key] = key < T ? (float)((s0[e] + s1[e]) * (double)inv_sqrt_dh) : -INFINITY;
  };
  // loads behind a condition would be waited for with the tile before them; a chunk past the end is the last one again
  fetch_k(0, min(wave, n_tiles - 1));
  __builtin_amdgcn_sched_barrier(0);
  fetch_k(1, min(wave + 4, n_tiles - 1));
  __builtin_amdgcn_sched_barrier(0);
  if (n_live && seq >= live) return;
  int kt = wave;
#pragma unroll 1
  for (; kt + 8 < n_tiles; kt += 8) {
    score(0, kt);
    fetch_k(0, kt + 8);
    score(1, kt + 4);
    fetch_k(1, min(kt + 12, n_tiles - 1));
  }
  if (kt < n_tiles) score(0, kt);
  if (kt + 4 < n_tiles) score(1, kt + 4);
  // values of the first kVRing tiles: on the way while the softmax runs
  constexpr int kVRing = 4;
  float vb[kVRing][4];
  auto fetch_v = [&](float *v, int dt, int kt) {
    kt = min(kt, n_tiles - 1);
    if constexpr (!WIN) {
#ifdef __HIP_DEVICE_COMPILE__
      const auto rs = rows_from(fresh + 2 * d + dt * 16 + (int64_t)kt * 16 * ld);
      const bool last = kt == n_tiles - 1;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, last ? v_last[e] : v_off[e], 0, 0));
#endif
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v_row(kt * 16 + 4 * fq + e)[dt * 16 + fr];
  };
  if (wave < KC) {
#pragma unroll
    for (int i = 0; i < kVRing; ++i) fetch_v(vb[i], wave, i);
  }
  __syncthreads();

  // ---- softmax over each row (the padding columns hold -inf, so their weight is 0): the wave's four rows side by side,
  // sixteen lanes each, because one row after the other is a chain of 12 shuffles a row.  A row is summed up as if its lanes
  // were a whole wave (keys k, k + 64, .. in one sum, then halves, quarters, ..). ----
  float *pr = s_p + (wave * 4 + fq) * stride;
  {
    float m = -INFINITY;
#pragma unroll 4
    for (int kt = 0; kt < n_tiles; ++kt) m = fmaxf(m, pr[kt * 16 + fr]);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float z[4] = {0.f, 0.f, 0.f, 0.f};
    int kt = 0;
    for (; kt + 4 <= n_tiles; kt += 4) {
      float e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = expf(pr[(kt + i) * 16 + fr] - m);
#pragma unroll
      for (int i = 0; i < 4; ++i) { pr[(kt + i) * 16 + fr] = e[i]; z[i] += e[i]; }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (kt + i < n_tiles) {
        const float e = expf(pr[(kt + i) * 16 + fr] - m);
        pr[(kt + i) * 16 + fr] = e; z[i] += e;
      }
    float t = (z[0] + z[2]) + (z[1] + z[3]);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o);
    const float inv = 1.0f / t;
    // multiplied here once, not by each of the four waves that read them
    for (kt = 0; kt + 8 <= n_tiles; kt += 8) {
      float e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = pr[(kt + i) * 16 + fr];
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[(kt + i) * 16 + fr] = e[i] * inv;
    }
    for (; kt < n_tiles; ++kt) pr[kt * 16 + fr] *= inv;
  }
  __syncthreads();

  // ---- out: row = query, column = lane % 16 of the wave's 16 columns ----
  for (int dt = wave; dt < KC; dt += 4) {
    doublex4 o0 = {0.0, 0.0, 0.0, 0.0}, o1 = o0;
    auto mul = [&](int buf, int kt) {
      if (kt * 16 + 16 > T) {                    // uniform: the weight of a padding column is 0, and 0 * inf would not be
#pragma unroll
        for (int e = 0; e < 4; ++e) vb[buf][e] = kt * 16 + 4 * fq + e < T ? vb[buf][e] : 0.f;
      }
      const float4 p = *reinterpret_cast<const float4 *>(s_p + fr * stride + kt * 16 + 4 * fq);
      o0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p.x, (double)vb[buf][0], o0, 0, 0, 0);
      o1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p.y, (double)vb[buf][1], o1, 0, 0, 0);
      o0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p.z, (double)vb[buf][2], o0, 0, 0, 0);
      o1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p.w, (double)vb[buf][3], o1, 0, 0, 0);
    };
    if (dt != wave) {
#pragma unroll
      for (int i = 0; i < kVRing; ++i) fetch_v(vb[i], dt, i);
    }
    for (int kt = 0; kt < n_tiles; kt += kVRing) {
#pragma unroll
      for (int i = 0; i < kVRing; ++i) {
        if (kt + i < n_tiles) mul(i, kt + i);
        fetch_v(vb[i], dt, kt + i + kVRing);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q_ = q0 + 4 * e + fq;
      if (q_ < n_rows) out[((int64_t)seq * n_rows + q_) * d + (int64_t)head * dh + dt * 16 + fr] = (float)(o0[e] + o1[e]);
    }
  }
}

size_t lds_bytes(int T) { return (size_t)TQ * ((T + 15) / 16 * 16 + 4) * sizeof(float); }

template <bool WIN>
pvf_status launch(pvf_ctx *ctx, hipStream_t s, const float *qkv, float *out, int S, int n_rows, int T, int n_heads, int d_head,
                  const WinF32 &wa, const int32_t *n_live = nullptr) {
  const size_t lds = lds_bytes(T);
  const dim3 grid((n_rows + TQ - 1) / TQ, n_heads, S);
  const float isd = 1.0f / sqrtf((float)d_head);
#define PVF_ATT_CASE(KC)                                                                                             \
  case KC: {                                                                                                         \
    static const hipError_t configured = hipFuncSetAttribute(reinterpret_cast<const void *>(attention_f32_kernel<KC, WIN>), \
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 64); \
    PVF_HIP_CHECK(ctx, configured);                                                                                  \
    attention_f32_kernel<KC, WIN><<<grid, 256, lds, s>>>(qkv, out, n_rows, T, n_heads, isd, n_live, wa);             \
    break;                                                                                                           \
  }
  switch (d_head / 16) {
    PVF_ATT_CASE(1) PVF_ATT_CASE(2) PVF_ATT_CASE(4) PVF_ATT_CASE(8)
    default: PVF_REQUIRE(ctx, false, PVF_ESHAPE, "attention_f32: d_head=%d", d_head);
  }
#undef PVF_ATT_CASE
  PVF_LAUNCH_CHECK(ctx, "attention_f32");
  return PVF_OK;
}

}  // namespace

bool attention_f32_supported(int dtype, int T, int d_head) {
  return dtype == PVF_F32 && (d_head == 16 || d_head == 32 || d_head == 64 || d_head == 128) && lds_bytes(T) <= 160 * 1024 - 64;
}

// qkv must already be rotated.
// n_live (may be NULL): device count of the canvases that are there, at most S.
pvf_status launch_attention_f32(pvf_ctx *ctx, hipStream_t s, const void *qkv, void *out, int S, int T, int n_heads, int d_head,
                                const int32_t *n_live) {
  if (S == 0) return PVF_OK;
  return launch<false>(ctx, s, (const float *)qkv, (float *)out, S, T, T, n_heads, d_head, WinF32{}, n_live);
}

pvf_status launch_attention_window_f32(pvf_ctx *ctx, hipStream_t s, const void *qkv_w, const void *kc, const void *vc,
                                       int64_t group_stride, const pvf_decode_cfg &cfg, const pvf_state &st,
                                       const int32_t *seq_slot, int n_seq, int n_heads, int d_head, void *out) {
  if (n_seq == 0) return PVF_OK;
  WinF32 wa;
  wa.kc = (const float *)kc; wa.vc = (const float *)vc; wa.group_stride = group_stride;
  wa.seq_slot = seq_slot; wa.k_active = st.k_active; wa.slots_per_group = 1 + cfg.K;
  wa.prompt_len = cfg.prompt_len; wa.block_len = cfg.block_len;
  return launch<true>(ctx, s, (const float *)qkv_w, (float *)out, n_seq, window_rows(cfg), cfg.prompt_len + cfg.gen_len, n_heads,
                      d_head, wa);
}

}  // namespace pvf
