// float32 GEMM with float64 sums on the matrix cores:  C[M,N] = A[M,K] * W[N,K]^T, any M, N, K, with the
// epilogues of the forward (store, + residual, SwiGLU, rotary embedding of the q and k thirds).  It is the
// float32 path: operands are widened to float64 in registers and multiplied by v_mfma_f64_16x16x4_f64, so a
// product is exact and a sum carries 53 bits, as on the plain kernel this replaces.
//
// What bounds it: in the small parity model latency (a launch of 384 rows is 0.2 GFLOP, 3 us of the chip's matrix rate, 78
// TFLOP/s in float64, behind 2.4 us that any launch takes), and from a few thousand rows on the SIMDs' issue: while a float64
// MFMA runs (64 cycles) its SIMD issues no vector instruction of any wave, so every one of them, the conversions of the operands
// above all, adds its 5 cycles to the MFMAs' (4 MFMAs with 4 conversions 71 TFLOP/s, with 16 float32 operations 60).  So
//   * operands go from global memory straight into registers in operand layout, with no LDS and no barrier
//     in the loop: a lane holds four consecutive k of its row (one 16-byte load) and feeds them to four MFMAs,
//     the contraction index being permuted alike on both operands.  The loads take a lane offset that stays and a scalar one
//     for k, which costs no vector instruction, and nothing is loaded that is not multiplied but for a chunk of waves with an odd
//     number of them: two chunks past the end, loaded so that the loop had no other form, cost 10 % at K = 256;
//   * the four waves of a workgroup share K, each taking every fourth 16-k chunk, and their tiles are added through LDS in wave
//     order.  Small launches get short loops that way, and large ones many equal workgroups.  The order in which an
//     element's k are added is the same for every tile shape, so a row's bits do not depend on the launch's size;
//   * tiles of 32 x 32, at most 128 registers: four workgroups a CU cover each other's prologue and epilogue, which are half of a
//     loop over 256 k.  64 x 32 tiles (three workgroups, a quarter fewer conversions) gain 4 % at 9160 rows of 4096 columns, nothing at
//     768 and lose at 256; workgroups that loop over tiles, the next one's loads behind the epilogue, lose 0-10 %.  SwiGLU
//     takes 32 rows x 16 gate and the same 16 up columns (32 + 32 columns need 230 registers: 108 -> 89 us);
//   * launches of few tiles take 16 rows where that leaves less to the fullest CU (run_epi);
//   * one or two chunks are on their way while another is multiplied, none behind a condition: the wait would then be for all of them.
// Measured on the small model's shapes, K = 256 but for the down projection's 704 (us per launch; plain vector-ALU kernel, loads by
// 64-bit addresses past the end too, now): QKV of 384 rows 42, 8.0, 6.9, of 4 580 rows 41 -> 38, of 9 160 75 -> 68 (53 TFLOP/s);
// gate/up of 384 rows 62, 10.9, 10.0, of 9 160 136 -> 121; down of 384 rows 81, 6.8, 6.5, of 916 11.5 -> 8.8; output head of 1 374 rows
// 63 -> 56, of 9 160 386 -> 329 (58 TFLOP/s; K = 4096 65 -> 69).
#include "common.h"

#include <algorithm>
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
  auto add = [&](int k0, auto n, auto whole) {                      // n loads on their way together
    constexpr int kN = decltype(n)::value;
    float4 v[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) v[i] = four<VEC>(x, k0 + 32 * i, K);
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const double q = ((double)v[i].x * v[i].x + (double)v[i].y * v[i].y) + ((double)v[i].z * v[i].z + (double)v[i].w * v[i].w);
      ss += decltype(whole)::value || k0 + 32 * i < K ? q : 0.0;
    }
  };
  // the first 256 outside of the loop, in front of which the compiler waits for every load on its way
  if (K >= 256) add(4 * j, std::integral_constant<int, 8>{}, std::true_type{});
#pragma unroll 1
  for (int k0 = K >= 256 ? 256 : 0; k0 < K; k0 += 128) add(k0 + 4 * j, std::integral_constant<int, 4>{}, std::false_type{});
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

// Orders LDS accesses of the workgroup without waiting for loads from global memory that are on their way.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// NORM: the operand is RMSNorm(A) * gain, each row's 1 / rms from float64 sums taken by the workgroup itself while its first
// chunks are on the way (and before it knows whether its rows are live: the count's load would stand in front of the rows'; rounds of
// 1-3 canvases x 128 tokens 4 % faster), the elements rounded to float32 as the norm's own pass rounds them.  MAP: rows through RowsF32::map.
// LOAD: kLoadAny element by element; otherwise 16 bytes through buffer descriptors, kLoadFour for K % 4 == 0, kLoadChunks for K % 16 == 0.
enum { kLoadAny, kLoadFour, kLoadChunks };
template <int EPI, int LOAD, bool NORM, bool MAP, int MT, int NT>
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
  const int n_chunks = (K + 15) / 16;
  const int tile_n = blockIdx.x % tiles_n, m0 = blockIdx.x / tiles_n * TM;

  auto src_row = [&](int m, bool *ok) -> int64_t {                  // row of A and Res behind row m
    *ok = true;
    if constexpr (!MAP) return m;
    const int s = m / rw.R, pos = rw.map[m];
    *ok = pos >= 0 && pos < rw.T;
    return (int64_t)s * rw.T + (*ok ? pos : 0);
  };
  const float *ap[MT], *wp[NB];                                     // kLoadAny
  uint32_t ao[MT], wo[NB];                                          // otherwise: byte offsets of the lane's four k in chunk 0
  const uint32_t tail_back = LOAD == kLoadFour ? 4u * max(0, (n_chunks - 1) * 16 + 4 * fq + 4 - K) : 0u;   // lanes past K: the row's last four
  bool a_ok[MT];
  // descriptors from the tile's own first rows of A and W on, so that a lane's offset has 32 bits whatever the matrix
  const int64_t first = MAP ? (int64_t)(m0 / rw.R) * rw.T : m0, n_src = MAP ? (int64_t)(M / rw.R) * rw.T : M;
  const int w_first = tile_col<EPI, TN>(tile_n, 0, ra.half);
#ifdef __HIP_DEVICE_COMPILE__                                       // the descriptor type does not exist in the host pass
  auto rows_from = [&](const float *x, int64_t row, int64_t rows) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)(x + row * K), 0, (int)(uint32_t)min((rows - row) * K * 4, (int64_t)0xfffffff0), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t rsA = rows_from(A, first, n_src), rsG = rows_from(rw.gain, 0, 1), rsW = rows_from(W, w_first, N);
  const __amdgpu_buffer_rsrc_t rsU = rows_from(W + (int64_t)(EPI == kEpiSwiglu ? N : 0) * K, w_first, N);      // SwiGLU: the up rows
#endif
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int64_t r = src_row(min(m0 + t * 16 + fr, M - 1), &a_ok[t]);           // ragged edge: a valid row again
    ap[t] = A + r * K;
    ao[t] = (uint32_t)(r - first) * (uint32_t)K * 4u + 16u * fq;
  }
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int n = min(tile_col<EPI, TN>(tile_n, (t % NT) * 16 + fr, ra.half), N - 1);
    wp[t] = W + (int64_t)(t >= NT ? N + n : n) * K;
    wo[t] = (uint32_t)(n - w_first) * (uint32_t)K * 4u + 16u * fq;
  }
  doublex4 acc[MT][NB];

  struct Chunk { float a[MT][4], w[NB][4], g[NORM ? 4 : 1]; };
  // 16 k from ch * 16.  The loads are unconditional (a chunk past the end is the last one again, and never multiplied), so that
  // the wait for a chunk lets the loads of the next one stay in flight; with the fetch behind a condition it waited for them all.
  auto fetch = [&](Chunk &c, int ch) {
    ch = min(ch, n_chunks - 1);
    if constexpr (LOAD == kLoadAny) {
      const int k = ch * 16 + 4 * fq;
      auto one = [&](const float *p, float *v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = k + e < K ? p[k + e] : 0.f;
      };
#pragma unroll
      for (int t = 0; t < MT; ++t) one(ap[t], c.a[t]);
#pragma unroll
      for (int t = 0; t < NB; ++t) one(wp[t], c.w[t]);
    } else {
#ifdef __HIP_DEVICE_COMPILE__
      const uint32_t back = LOAD == kLoadFour && ch == n_chunks - 1 ? tail_back : 0u;
      auto one = [&](__amdgpu_buffer_rsrc_t rs, uint32_t o, float *v) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rs, LOAD == kLoadFour ? o - back : o, ch * 64, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(x[e]);
      };
#pragma unroll
      for (int t = 0; t < MT; ++t) one(rsA, ao[t], c.a[t]);
#pragma unroll
      for (int t = 0; t < NB; ++t) one(t >= NT ? rsU : rsW, wo[t], c.w[t]);
      if constexpr (NORM) one(rsG, 16u * fq, c.g);
#endif
    }
  };
  float rnorm[MT];
  auto multiply = [&](Chunk &c, int ch) {
    if (LOAD == kLoadFour && ch == n_chunks - 1) {                  // uniform: lanes past K bring nothing
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
    for (int e = 0; e < 4; ++e) {
      double w[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) w[j] = (double)c.w[j][e];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        float a = c.a[i][e];
        if constexpr (NORM) a = a * rnorm[i] * c.g[NORM ? e : 0];
        if (MAP && !a_ok[i]) a = 0.f;
        const double ad = (double)a;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad, w[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  __shared__ double part[WK][MT * NB][4][64];
  __shared__ float s_r[NORM ? TM : 1];
  Chunk c0, c1;
  fetch(c0, wave);
  __builtin_amdgcn_sched_barrier(0);                                // one chunk's loads behind the other's
  fetch(c1, wave + WK);
  __builtin_amdgcn_sched_barrier(0);
  // uniform; the count is asked for beside the loads, not in front of them
  const int live = rw.n_live ? *rw.n_live : 0;
  if constexpr (NORM) {
    const int row = threadIdx.x >> 3, j = threadIdx.x & 7;          // eight threads a row
    float r = 0.f;
    if (row < TM) r = row_rnorm(A + (int64_t)min(m0 + row, M - 1) * K, j, K, rw.inv_k, rw.eps);
    if (rw.n_live && m0 >= live * rw.per_seq) return;
    if (row < TM && j == 0) s_r[row] = r;
    lds_barrier();
#pragma unroll
    for (int t = 0; t < MT; ++t) rnorm[t] = s_r[t * 16 + fr];
  } else if (rw.n_live && m0 >= live * rw.per_seq) return;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  // this wave's chunks: one or two on their way while another is multiplied
  int ch = wave;
#pragma unroll 1
  for (; ch + 2 * WK < n_chunks; ch += 2 * WK) {
    multiply(c0, ch);
    fetch(c0, ch + 2 * WK);
    multiply(c1, ch + WK);
    fetch(c1, ch + 3 * WK);
  }
  if (ch < n_chunks) multiply(c0, ch);
  if (ch + WK < n_chunks) multiply(c1, ch + WK);
  // ---- wave w adds up register w of every tile (rows 4 w + lane / 16) over the four waves, in wave order ----
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][i * NB + j][e][lane] = acc[i][j][e];
  lds_barrier();
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
  const bool aligned = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)rw.gain) & 15u) == 0;
  // the rows of a tile, of a head, or of the canvases that a tile's rows are picked from lie within 32-bit offsets
  const bool vec = aligned && std::max<int64_t>(256, MAP ? ((int64_t)32 / std::max(rw.R, 1) + 2) * rw.T : 0) * K * 4 < (1ll << 32);
  auto launch = [&](auto mt, auto nt) -> pvf_status {
    constexpr int MT = decltype(mt)::value, NT = decltype(nt)::value;
    const int64_t tiles = (int64_t)((N + 16 * NT - 1) / (16 * NT)) * ((M + 16 * MT - 1) / (16 * MT));
    PVF_REQUIRE(ctx, tiles < (1ll << 31), PVF_ESHAPE, "gemm_f32: M=%d N=%d", M, N);
    const unsigned grid = (unsigned)tiles;
    if (vec && K % 16 == 0) gemm_f32_kernel<EPI, kLoadChunks, NORM, MAP, MT, NT><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra, rw);
    else if (vec) gemm_f32_kernel<EPI, kLoadFour, NORM, MAP, MT, NT><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra, rw);
    else if constexpr (!NORM) gemm_f32_kernel<EPI, kLoadAny, NORM, MAP, MT, NT><<<grid, 256, 0, s>>>(A, W, C, res, M, N, K, ra, rw);
    else PVF_REQUIRE(ctx, false, PVF_ESHAPE, "gemm_f32: the fused norm takes 16-byte aligned rows of less than 4M elements");
    PVF_LAUNCH_CHECK(ctx, "gemm_f32");
    return PVF_OK;
  };
  using std::integral_constant;
  constexpr integral_constant<int, 1> k1{};
  constexpr integral_constant<int, 2> k2{};
  constexpr integral_constant<int, EPI == kEpiSwiglu ? 1 : 2> nt{};
  // 16 or 32 rows a tile by workgroups on the fullest CU: one of 16 rows takes 1.5 us of a CU's matrix units at K = 256 and one of 32
  // rows 2.5 (4.2 and 6.5 at K = 704).  K = 256, QKV of 768 columns: 384 rows 6.8 us (16) and 7.5 (32), 576 rows 8.5 and 7.7, 1145 rows
  // 12.9 and 12.5; gate/up of 704: 64 rows 3.9 and 5.2, 160 rows 5.5 and 5.4, 384 rows 10.0 and 10.5, 687 rows 14.3 and 12.8.  K = 704, 256
  // columns: 512 rows 6.5 and 8.8, 576 rows 10.7 and 8.7, 2290 rows 23.1 and 21.9.
  const int64_t cols = (N + 16 * decltype(nt)::value - 1) / (16 * decltype(nt)::value);
  const int64_t c1 = (cols * ((M + 15) / 16) + 255) / 256, c2 = (cols * ((M + 31) / 32) + 255) / 256;
  return (K <= 512 ? 3 * c1 <= 5 * c2 : 2 * c1 <= 3 * c2) ? launch(k1, nt) : launch(k2, nt);
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
