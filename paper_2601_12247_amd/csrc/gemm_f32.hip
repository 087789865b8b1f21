// float32 GEMM with float64 sums on the matrix cores:  C[M,N] = A[M,K] * W[N,K]^T, any M, N, K, with the
// epilogues of the forward (store, + residual, SwiGLU, rotary embedding of the q and k thirds).  It is the
// float32 path: operands are widened to float64 in registers and multiplied by v_mfma_f64_16x16x4_f64, so a
// product is exact and a sum carries 53 bits, as on the plain kernel this replaces.
//
// What bounds it: in the small parity model latency -- a launch of 384 rows is 0.2 GFLOP, 3 us of the chip's
// matrix rate (78 TFLOP/s in float64) -- and from a few thousand rows on that rate.  So
//   * operands go from global memory straight into registers in operand layout, with no LDS and no barrier
//     in the loop: a lane holds four consecutive k of its row (one 16-byte load) and feeds them to four MFMAs,
//     the contraction index being permuted alike on both operands;
//   * the four waves of a workgroup share K, each taking every fourth 16-k chunk, and their tiles are added through LDS in wave
//     order.  Small launches get short loops that way, and large ones many equal workgroups.  The order in which an
//     element's k are added is the same for every tile shape, so a row's bits do not depend on the launch's size;
//   * tiles of 32 x 32, at most 128 registers: four workgroups a CU instead of three cover each other's
//     prologue and epilogue, which are half of a loop over 256 k (6 236 rows: QKV 60 -> 52 us, down projection 57 -> 52).  SwiGLU
//     takes 32 rows x 16 gate and the same 16 up columns for the same reason (32 + 32 columns need 230 registers: 108 -> 89 us);
//   * launches of at most 512 such tiles (two a CU) take 16 x 32 instead: twice as many workgroups with
//     half the work each (384 rows: QKV 9.7 -> 8.2 us, down 12.1 -> 7.9; above, the bigger tile reads less: 52 against 62 us);
//   * one or two chunks are on their way while another is multiplied (one chunk ahead, fetched under a condition, every chunk was
//     waited for whole; with that and the rows of the fused norm read eight loads at a time, rounds of 1-3 canvases x 128
//     tokens 131 -> 120 us, of 8-40 canvases x 229 539 -> 525).
// Measured on the small model's shapes (us per launch, plain vector-ALU kernel -> this one): QKV of 384 rows 42 -> 8, gate/up
// 62 -> 11, down 81 -> 8; gate/up of 6 236 rows 89 (50 TFLOP/s), output head of 1 743 rows 75 (49 TFLOP/s).
#include "common.h"

#include <type_traits>

namespace pvf {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double silu_f64(double g) { return g / (1.0 + exp(-g)); }

// Four consecutive elements from k of a row of K; past its end zeros (VEC: the row's last four, which the caller leaves out).
template <bool VEC>
__device__ __forceinline__ float4 four(const float *x, int k, int K) {
  if constexpr (VEC) return *reinterpret_cast<const float4 *>(x + min(k, K - 4));
  auto one = [&](int i) { const float v = x[min(i, K - 1)]; return i < K ? v : 0.f; };
  return make_float4(one(k), one(k + 1), one(k + 2), one(k + 3));
}

// 1 / rms of a row that eight neighbouring threads share (j = 0..7), from float64 sums; every one of them gets it.  The fused
// norm and the pass of its own take it from here, at any alignment and in window rows too, so that which of them a launch takes
// does not show in a bit.  (Rows longer than kNormF32Max have one norm as well, rmsnorm_kernel.)
template <bool VEC = true>
__device__ __forceinline__ float row_rnorm(const float *x, int j, int K, double inv_k, float eps) {
  double ss = 0.0;
  for (int k0 = 4 * j; k0 < K; k0 += 256) {                         // eight loads on their way together
    float4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = four<VEC>(x, k0 + 32 * i, K);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (k0 + 32 * i < K)
        ss += ((double)v[i].x * v[i].x + (double)v[i].y * v[i].y) + ((double)v[i].z * v[i].z + (double)v[i].w * v[i].w);
  }
  ss += __shfl_xor(ss, 1); ss += __shfl_xor(ss, 2); ss += __shfl_xor(ss, 4);
  // the hardware's estimate of 1 / sqrt (relative error below 2^-22) and one Newton step, 1.5 times its square: below 2^-43, in a
  // tenth of the instructions of sqrt and divide
  const double v = ss * inv_k + (double)eps, r = __builtin_amdgcn_rsq(v);
  return (float)(r * fma(-0.5 * v * r, r, 1.5));
}

// out = RMSNorm(x) * gain, eight threads a row.  VEC: 16-byte loads, K % 4 == 0.
template <bool VEC>
__global__ void __launch_bounds__(256)
rmsnorm_f32_kernel(const float *__restrict__ x, const float *__restrict__ gain, float *__restrict__ out, int M, int K, double inv_k, float eps,
                   const int32_t *__restrict__ n_live, int per_seq) {
  const int m = blockIdx.x * 32 + (threadIdx.x >> 3), j = threadIdx.x & 7;
  if (n_live) M = min(M, *n_live * per_seq);
  if (m >= M) return;                                               // whole rows, so whole groups of eight
  const float *xr = x + (int64_t)m * K;
  const float r = row_rnorm<VEC>(xr, j, K, inv_k, eps);
#pragma unroll 4
  for (int k = 4 * j; k < K; k += 32) {
    const float4 v = four<VEC>(xr, k, K), g = four<VEC>(gain, k, K);
    const float4 o = make_float4(v.x * r * g.x, v.y * r * g.y, v.z * r * g.z, v.w * r * g.w);
    float *to = out + (int64_t)m * K + k;
    if constexpr (VEC) { *reinterpret_cast<float4 *>(to) = o; continue; }
    const float e[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) if (k + i < K) to[i] = e[i];
  }
}

// W row behind column c (0..31) of a 32-column wave tile: with the rotary epilogue the second 16 columns are the
// rotation partners (+ d_head / 2) of the first 16, so that a pair meets in one lane.
template <int EPI, int TN>
__device__ __forceinline__ int tile_col(int tile, int c, int half) {
  if (EPI != kEpiQkvRope) return tile * TN + c;
  const int per_head = half / 16;                                   // wave tiles per head
  const int head = tile / per_head, j = tile % per_head;
  return head * 2 * half + j * 16 + (c >= 16 ? half : 0) + (c & 15);
}

// NORM: the operand is RMSNorm(A) * gain, each row's 1 / rms from float64 sums taken by the workgroup itself while its first
// chunks are on the way, the elements rounded to float32 as the norm's own pass rounds them.  MAP: rows through RowsF32::map.
template <int EPI, bool VEC, bool NORM, bool MAP, int MT, int NT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8)))
gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W, float *__restrict__ C,
                const float *__restrict__ Res, int M, int N, int K, RopeF32 ra, RowsF32 rw) {
  constexpr int WK = 4;                                             // waves that share K
  constexpr int TM = 16 * MT, TN = 16 * NT;
  static_assert(EPI != kEpiQkvRope || NT == 2, "a rotation pair is two tiles wide");
  constexpr int NB = EPI == kEpiSwiglu ? 2 * NT : NT;               // SwiGLU: gate tiles, then up tiles
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fq = lane >> 4;
  const int tiles_n = (N + TN - 1) / TN;
  const int tile_n = blockIdx.x % tiles_n, m0 = blockIdx.x / tiles_n * TM;

  auto src_row = [&](int m, bool *ok) -> int64_t {                  // row of A and Res behind row m
    *ok = true;
    if constexpr (!MAP) return m;
    const int s = m / rw.R, pos = rw.map[m];
    *ok = pos >= 0 && pos < rw.T;
    return (int64_t)s * rw.T + (*ok ? pos : 0);
  };
  const float *ap[MT], *wp[NB], *gp = rw.gain;
  bool a_ok[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) ap[t] = A + src_row(min(m0 + t * 16 + fr, M - 1), &a_ok[t]) * K;   // ragged edge: a valid row again
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int n = min(tile_col<EPI, TN>(tile_n, (t % NT) * 16 + fr, ra.half), N - 1);
    wp[t] = W + (int64_t)(t >= NT ? N + n : n) * K;
  }
  doublex4 acc[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

  struct Chunk { float a[MT][4], w[NB][4], g[NORM ? 4 : 1]; };
  const int n_chunks = (K + 15) / 16;
  // 16 k from ch * 16.  The loads are unconditional (a chunk past the end is the last one again, and never multiplied), so that
  // the wait for a chunk lets the loads of the next one stay in flight; with the fetch behind a condition it waited for them all.
  auto fetch = [&](Chunk &c, int ch) {
    const int k = min(ch, n_chunks - 1) * 16 + 4 * fq;
    const int kv = VEC ? min(k, K - 4) : k;
    auto one = [&](const float *p, float *v) {
      if (VEC) {
        const float4 x = *reinterpret_cast<const float4 *>(p + kv);
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
    if constexpr (NORM) one(gp, c.g);
  };
  float rnorm[MT];
  auto multiply = [&](Chunk &c, int ch) {
    if (VEC && K % 16 != 0 && ch == n_chunks - 1) {                 // uniform: lanes past K bring nothing
      const bool in = ch * 16 + 4 * fq < K;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int t = 0; t < MT; ++t) c.a[t][e] = in ? c.a[t][e] : 0.f;
#pragma unroll
        for (int t = 0; t < NB; ++t) c.w[t][e] = in ? c.w[t][e] : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        float a = c.a[i][e];
        if constexpr (NORM) a = a * rnorm[i] * c.g[NORM ? e : 0];
        if (MAP && !a_ok[i]) a = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a, (double)c.w[j][e], acc[i][j], 0, 0, 0);
      }
  };
  // this wave's chunks wave, wave + 4, ...: one or two on their way while another is multiplied
  Chunk c0, c1;
  fetch(c0, wave);
  fetch(c1, wave + WK);
  if (rw.n_live && m0 >= *rw.n_live * rw.per_seq) return;           // uniform
  if constexpr (NORM) {
    __shared__ float s_r[TM];
    const int row = threadIdx.x >> 3, j = threadIdx.x & 7;          // eight threads a row
    if (row < TM) {
      const float r = row_rnorm(A + (int64_t)min(m0 + row, M - 1) * K, j, K, rw.inv_k, rw.eps);
      if (j == 0) s_r[row] = r;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MT; ++t) rnorm[t] = s_r[t * 16 + fr];
  }
#pragma unroll 1
  for (int ch = wave; ch < n_chunks; ch += 2 * WK) {
    multiply(c0, ch);
    fetch(c0, ch + 2 * WK);
    if (ch + WK < n_chunks) multiply(c1, ch + WK);
    fetch(c1, ch + 3 * WK);
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
    bool r_ok = true;
    const float *rrow = EPI == kEpiResidual ? Res + src_row(m, &r_ok) * N : nullptr;
    if (EPI == kEpiQkvRope) {
      const int n = tile_col<EPI, TN>(tile_n, fr, ra.half);           // and its partner n + half; N = 3 d is a whole number of heads
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
      const int n = tile_n * TN + j * 16 + fr;
      if (n >= N) continue;
      double x = v[i][j];
      if (EPI == kEpiResidual && r_ok) x += (double)rrow[n];
      if (EPI == kEpiSwiglu) x = silu_f64(x) * v[i][NT + j];
      row[n] = (float)x;
    }
  }
}

template <int EPI, bool NORM = false, bool MAP = false>
pvf_status run_epi(pvf_ctx *ctx, hipStream_t s, const float *A, const float *W, float *C, const float *res, int M, int N, int K,
                   const RopeF32 &ra, const RowsF32 &rw = RowsF32{}) {
  const bool vec = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)rw.gain) & 15u) == 0;
  auto launch = [&](auto mt, auto nt) -> pvf_status {
    constexpr int MT = decltype(mt)::value, NT = decltype(nt)::value;
    const int64_t tiles = (int64_t)((N + 16 * NT - 1) / (16 * NT)) * ((M + 16 * MT - 1) / (16 * MT));
    PVF_REQUIRE(ctx, tiles < (1ll << 31), PVF_ESHAPE, "gemm_f32: M=%d N=%d", M, N);
    const unsigned grid = (unsigned)tiles;
    if (vec) gemm_f32_kernel<EPI, true, NORM, MAP, MT, NT><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra, rw);
    else if constexpr (!NORM) gemm_f32_kernel<EPI, false, NORM, MAP, MT, NT><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra, rw);
    else PVF_REQUIRE(ctx, false, PVF_ESHAPE, "gemm_f32: the fused norm takes 16-byte aligned rows");
    PVF_LAUNCH_CHECK(ctx, "gemm_f32");
    return PVF_OK;
  };
  using std::integral_constant;
  constexpr integral_constant<int, 1> k1{};
  constexpr integral_constant<int, 2> k2{};
  const int64_t tiles32 = (int64_t)((N + 31) / 32) * ((M + 31) / 32);
  if constexpr (EPI == kEpiSwiglu) return launch(k2, k1);
  else return tiles32 <= 512 ? launch(k1, k2) : launch(k2, k2);
}

}  // namespace

pvf_status launch_gemm_f32(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const float *A, const float *W, float *C,
                           const float *res, int M, int N, int K, const RowsF32 *rows) {
  if (M == 0 || N == 0) return PVF_OK;
  const RopeF32 none{};
  const RowsF32 rw = rows ? *rows : RowsF32{};
  switch (epi) {
    case kEpiStore: return rw.gain ? run_epi<kEpiStore, true>(ctx, s, A, W, C, res, M, N, K, none, rw) : run_epi<kEpiStore>(ctx, s, A, W, C, res, M, N, K, none, rw);
    case kEpiResidual: return rw.map ? run_epi<kEpiResidual, false, true>(ctx, s, A, W, C, res, M, N, K, none, rw) : run_epi<kEpiResidual>(ctx, s, A, W, C, res, M, N, K, none, rw);
    case kEpiSwiglu: return rw.gain ? run_epi<kEpiSwiglu, true>(ctx, s, A, W, C, res, M, N, K, none, rw) : run_epi<kEpiSwiglu>(ctx, s, A, W, C, res, M, N, K, none, rw);
    default: PVF_REQUIRE(ctx, false, PVF_ENOTIMPL, "gemm_f32: epilogue %d has its own entry", (int)epi);
  }
}

// Whether the projections that read a normed stream of rows d long take the norm along.  Every workgroup of a row of tiles
// norms the same rows again, half as many bytes once more as its main loop reads, which costs less than a launch and a pass
// where rows and launches are short (1-3 canvases x 128 tokens, 256 wide: a round with five norms 157 -> 136 us) and more where
// there are many rows (8 canvases x 229 with drafts: 565 -> 612): fused up to 1280 rows (forward_f32_impl).
bool gemm_f32_norm_supported(int d) { return d <= kNormF32Max && d % 4 == 0; }

pvf_status launch_rmsnorm_f32(pvf_ctx *ctx, hipStream_t s, const float *x, float *out, int M, int K, const RowsF32 &rows) {
  if (M == 0) return PVF_OK;
  const bool vec = K % 4 == 0 && (((uintptr_t)x | (uintptr_t)rows.gain | (uintptr_t)out) & 15u) == 0;
  (vec ? rmsnorm_f32_kernel<true> : rmsnorm_f32_kernel<false>)<<<(M + 31) / 32, 256, 0, s>>>(x, rows.gain, out, M, K, rows.inv_k, rows.eps,
                                                                                            rows.n_live, rows.per_seq);
  PVF_LAUNCH_CHECK(ctx, "rmsnorm_f32");
  return PVF_OK;
}

// QKV projection whose epilogue rotates q and k: qkv[M, 3 d] with d_head % 32 == 0.
bool gemm_f32_qkv_rope_supported(int d_head) { return d_head % 32 == 0; }

pvf_status launch_gemm_f32_qkv_rope(pvf_ctx *ctx, hipStream_t s, const float *A, const float *W, float *qkv, int M, int d, int K,
                                    const RopeF32 &ra, const RowsF32 *rows) {
  if (M == 0) return PVF_OK;
  if (rows && rows->gain) return run_epi<kEpiQkvRope, true>(ctx, s, A, W, qkv, nullptr, M, 3 * d, K, ra, *rows);
  return run_epi<kEpiQkvRope>(ctx, s, A, W, qkv, nullptr, M, 3 * d, K, ra, rows ? *rows : RowsF32{});
}

}  // namespace pvf
