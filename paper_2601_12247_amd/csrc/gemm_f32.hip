// float32 GEMM with float64 sums on the matrix cores:  C[M,N] = A[M,K] * W[N,K]^T, any M, N, K, with the
// epilogues of the forward (store, + residual, SwiGLU, rotary embedding of the q and k thirds).  It is the
// float32 path: operands are widened to float64 in registers and multiplied by v_mfma_f64_16x16x4_f64, so a
// product is exact and a sum carries 53 bits, as on the plain kernel this replaces.
//
// What bounds it: in the small parity model latency -- a launch of 384 rows is 0.2 GFLOP, 3 us of the chip's
// matrix rate (78 TFLOP/s in float64) -- and from a few thousand rows on that rate.  So
//   * operands go from global memory straight into registers in operand layout, with no LDS and no barrier
//     in the loop: a lane holds four consecutive k of its row (one 16-byte load) and feeds them to four MFMAs,
//     the contraction index being permuted alike on both operands.  Two 16-k chunks are in flight per wave;
//   * a workgroup computes a 32 x 32 tile (SwiGLU: 32 gate and the same 32 up columns); its four waves share K, each
//     taking every fourth chunk, and their tiles are added through LDS in wave order.  Small launches get short
//     loops that way, and large ones many equal workgroups: 64 x 64 tiles with a quarter per wave and K undivided
//     were 0-30 % slower at 4 580 - 9 160 rows (they leave the last wave of workgroups emptier) and 5 % faster only
//     where N = 4096.
// Measured on the small model's shapes (us per launch, plain kernel -> this one): QKV of 384 rows 42 -> 10, gate/up
// 62 -> 17, down 81 -> 12; gate/up of 9 160 rows 148 (44 TFLOP/s), output head 395 (49 TFLOP/s).
#include "common.h"

namespace pvf {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double silu_f64(double g) { return g / (1.0 + exp(-g)); }

// W row behind column c (0..31) of a 32-column wave tile: with the rotary epilogue the second 16 columns are the
// rotation partners (+ d_head / 2) of the first 16, so that a pair meets in one lane.
template <int EPI>
__device__ __forceinline__ int tile_col(int tile, int c, int half) {
  if (EPI != kEpiQkvRope) return tile * 32 + c;
  const int per_head = half / 16;                                   // wave tiles per head
  const int head = tile / per_head, j = tile % per_head;
  return head * 2 * half + j * 16 + (c >= 16 ? half : 0) + (c & 15);
}

template <int EPI, bool VEC>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W, float *__restrict__ C,
                const float *__restrict__ Res, int M, int N, int K, RopeF32 ra) {
  constexpr int MT = 2, NT = 2, WK = 4;                             // 16 x 16 tiles in each direction; waves that share K
  constexpr int NB = EPI == kEpiSwiglu ? 2 * NT : NT;               // SwiGLU: gate tiles, then up tiles
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, fq = lane >> 4;
  const int tiles_n = (N + 31) / 32;
  const int tile_n = blockIdx.x % tiles_n, m0 = blockIdx.x / tiles_n * 32;

  const float *ap[MT], *wp[NB];
#pragma unroll
  for (int t = 0; t < MT; ++t) ap[t] = A + (int64_t)min(m0 + t * 16 + fr, M - 1) * K;   // ragged edge: a valid row again
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int n = min(tile_col<EPI>(tile_n, (t % NT) * 16 + fr, ra.half), N - 1);
    wp[t] = W + (int64_t)(t >= NT ? N + n : n) * K;
  }
  doublex4 acc[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

  struct Chunk { float a[MT][4], w[NB][4]; };
  const int n_chunks = (K + 15) / 16;
  auto fetch = [&](Chunk &c, int ch) {                              // 16 k from ch * 16; lanes past K hold zeros
    const int k = ch * 16 + 4 * fq;
    auto one = [&](const float *p, float *v) {
      if (VEC) {
        const float4 x = k < K ? *reinterpret_cast<const float4 *>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = k + e < K ? p[k + e] : 0.f;
      }
    };
#pragma unroll
    for (int t = 0; t < MT; ++t) one(ap[t], c.a[t]);
#pragma unroll
    for (int t = 0; t < NB; ++t) one(wp[t], c.w[t]);
  };
  auto multiply = [&](const Chunk &c) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)c.a[i][e], (double)c.w[j][e], acc[i][j], 0, 0, 0);
  };
  // this wave's chunks wave, wave + 4, ...: two in registers ahead of the one being multiplied.  (One call of multiply: with
  // the loop unrolled over the buffers the accumulators were copied between register files at every turn.)
  Chunk c0, c1, c2;
  fetch(c0, wave);
  fetch(c1, wave + WK);
#pragma unroll 1
  for (int ch = wave; ch < n_chunks; ch += WK) {
    fetch(c2, ch + 2 * WK);
    multiply(c0);
    c0 = c1; c1 = c2;
  }

  // ---- wave w adds up register w of every tile (rows 4 w + lane / 16) over the four waves, in wave order ----
  __shared__ double part[WK][MT * NB][4][64];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][i * NB + j][e][lane] = acc[i][j][e];
  __syncthreads();
  double v[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int t = i * NB + j;
      v[i][j] = ((part[0][t][wave][lane] + part[1][t][wave][lane]) + part[2][t][wave][lane]) + part[3][t][wave][lane];
    }
  // ---- epilogue: row 4 wave + lane / 16, column lane % 16 of each tile ----
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + i * 16 + 4 * wave + fq;
    if (m >= M) continue;
    float *row = C + (int64_t)m * N;
    if (EPI == kEpiQkvRope) {
      const int n = tile_col<EPI>(tile_n, fr, ra.half);           // and its partner n + half; N = 3 d is a whole number of heads
      if (n >= N) continue;
      const float a = (float)v[i][0], b = (float)v[i][1];
      if (n < 2 * (N / 3)) {
        const int64_t pos = ra.row_pos ? (ra.row_pos[m] < 0 ? ra.T - 1 : ra.row_pos[m]) : m % ra.T;
        const float2 cs = ra.cos_sin[pos * ra.half + n % (2 * ra.half)];
        row[n] = a * cs.x - b * cs.y;
        row[n + ra.half] = b * cs.x + a * cs.y;
      } else {
        row[n] = a;
        row[n + ra.half] = b;
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n = tile_n * 32 + j * 16 + fr;
      if (n >= N) continue;
      double x = v[i][j];
      if (EPI == kEpiResidual) x += (double)Res[(int64_t)m * N + n];
      if (EPI == kEpiSwiglu) x = silu_f64(x) * v[i][NT + j];
      row[n] = (float)x;
    }
  }
}

template <int EPI>
pvf_status run_epi(pvf_ctx *ctx, hipStream_t s, const float *A, const float *W, float *C, const float *res, int M, int N, int K,
                   const RopeF32 &ra) {
  const bool vec = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15u) == 0;
  const int64_t tiles = (int64_t)((N + 31) / 32) * ((M + 31) / 32);
  PVF_REQUIRE(ctx, tiles < (1ll << 31), PVF_ESHAPE, "gemm_f32: M=%d N=%d", M, N);
  const unsigned grid = (unsigned)tiles;
  if (vec) gemm_f32_kernel<EPI, true><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra);
  else gemm_f32_kernel<EPI, false><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra);
  PVF_LAUNCH_CHECK(ctx, "gemm_f32");
  return PVF_OK;
}

}  // namespace

pvf_status launch_gemm_f32(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const float *A, const float *W, float *C,
                           const float *res, int M, int N, int K) {
  if (M == 0 || N == 0) return PVF_OK;
  const RopeF32 none{};
  switch (epi) {
    case kEpiStore: return run_epi<kEpiStore>(ctx, s, A, W, C, res, M, N, K, none);
    case kEpiResidual: return run_epi<kEpiResidual>(ctx, s, A, W, C, res, M, N, K, none);
    case kEpiSwiglu: return run_epi<kEpiSwiglu>(ctx, s, A, W, C, res, M, N, K, none);
    default: PVF_REQUIRE(ctx, false, PVF_ENOTIMPL, "gemm_f32: epilogue %d has its own entry", (int)epi);
  }
}

// QKV projection whose epilogue rotates q and k: qkv[M, 3 d] with d_head % 32 == 0.
bool gemm_f32_qkv_rope_supported(int d_head) { return d_head % 32 == 0; }

pvf_status launch_gemm_f32_qkv_rope(pvf_ctx *ctx, hipStream_t s, const float *A, const float *W, float *qkv, int M, int d, int K,
                                    const RopeF32 &ra) {
  if (M == 0) return PVF_OK;
  return run_epi<kEpiQkvRope>(ctx, s, A, W, qkv, nullptr, M, 3 * d, K, ra);
}

}  // namespace pvf
