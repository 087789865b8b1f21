// Decision epilogue of a PVF round.
//
// stage 1  one pass over every live logits row: top-1 token (lowest id on ties, the [MASK]
//          column excluded) and its softmax probability (Sec. 3, definitions of y-hat and p).
//          The row is streamed once from HBM with 16-byte loads; the softmax itself is never
//          written anywhere.  Calibration takes the row's entropy in the same pass (float64 sums).
// stage 2 (the decisions on those summaries) lives in decision.hip.
#include "common.h"

#include <math.h>

#include <type_traits>

namespace pvf {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegInf = -INFINITY;
constexpr float kLog2eLo = 1.9259629911266174e-08f;     // log2 e - kLog2e

__device__ __forceinline__ float mul_rn(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// Sums of two float64 values over a wave
__device__ __forceinline__ void wave_sum2(double &a, double &b) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, kWave);
    b += __shfl_xor(b, o, kWave);
  }
}

// 2^x by the hardware instruction (no denormal fix-up: results below 2^-126 flush to 0).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ------------------------------------------------------------------------------------
// stage 1
// ------------------------------------------------------------------------------------
template <typename T> struct Vec16;  // how a 16-byte load splits into elements
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  static constexpr uint32_t kFill = 0xff80ff80u;  // two bf16 -inf
  __device__ static __forceinline__ void unpack(const uint4 &w, float *f) {
    f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
    f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
    f[4] = __uint_as_float(w.z << 16); f[5] = __uint_as_float(w.z & 0xffff0000u);
    f[6] = __uint_as_float(w.w << 16); f[7] = __uint_as_float(w.w & 0xffff0000u);
  }
};
template <> struct Vec16<float> {
  static constexpr int N = 4;
  static constexpr uint32_t kFill = 0xff800000u;  // -inf
  __device__ static __forceinline__ void unpack(const uint4 &w, float *f) {
    f[0] = __uint_as_float(w.x); f[1] = __uint_as_float(w.y);
    f[2] = __uint_as_float(w.z); f[3] = __uint_as_float(w.w);
  }
};

// 16-byte load with the non-temporal hint: a logits row is read exactly once, so it should not
// displace anything in the caches (measured: 6.5 instead of 5.9 TB/s on 2048 full-width rows).
__device__ __forceinline__ uint4 load_stream(const uint4 *p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}

// log2(e) (times the logit scale) as the sum of two floats, the second above zero: an infinite t below the max then gives
// t * hi + t * lo = -inf and not a NaN.
struct Log2e {
  float hi, lo;
  __device__ __forceinline__ explicit Log2e(float scale) {
    hi = scale * kLog2e;
    lo = fmaf(scale, kLog2e, -hi) + scale * kLog2eLo;
    if (!(lo > 0.f)) {
      hi = __uint_as_float(__float_as_uint(hi) - 1);
      lo = fmaf(scale, kLog2e, -hi) + scale * kLog2eLo;
    }
  }
  __device__ __forceinline__ float exp(float t) const { return fast_exp2(fmaf(t, lo, t * hi)); }
};

// Running (max, sum of exponentials) of one thread.  Values v live in the "compare domain": the raw
// logit for bf16 rows (scaling by a positive factor keeps order and ties of bf16 values; differences of bf16 values are
// exact), or logit_scale * logit for float rows.
//   fine:  terms 2^((v - m) c) with c in two parts, and what adding a group to the sum rounds off kept beside it: conf is
//          1e-10 (one-hot rows) to 2e-7 (many small terms beside a large one) from float64.
//   plain: terms 2^(v*c + nmc) with nmc = -fl(m*c), three instructions fewer; every term of the thread is therefore off by
//          the same factor 2^delta, delta = m*c - fl(m*c), which is known exactly and divided out when the thread's sum is
//          handed on: 7e-8 to 3e-7 from float64.
// Aligned rows of 4096 vectors and more keep the plain terms: the instructions of the fine ones show there (16 rows of 126464
// bf16 10.4 -> 13.2 us, 1190 rows of 50264 23.3 -> 25.0).  All others take the fine ones and wait for memory all the same.
template <bool kFine> struct Running;
template <> struct Running<true> {
  const Log2e c;
  float m = kNegInf, z = 0.f, zc = 0.f;
  int first = INT_MAX, cnt = 0;      // vectors first, first+BLOCK, .. (cnt of them) held the value that raised m; cnt = 0: element first
  __device__ __forceinline__ explicit Running(float scale) : c(scale) {}
  __device__ __forceinline__ void raise(float gm, int first_vec, int n_vec) {
    if (m > kNegInf) { const float f = c.exp(m - gm); z *= f; zc *= f; }
    m = gm; first = first_vec; cnt = n_vec;
  }
  __device__ __forceinline__ float term(float v) const { return c.exp(v - m); }
  __device__ __forceinline__ void add(float a) {
    const float s = z + a, b = s - z;
    zc += (z - (s - b)) + (a - b);
    z = s;
  }
  __device__ __forceinline__ float sum_for(float M) const { return (z + zc) * c.exp(m - M); }     // relative to M >= m
};
template <> struct Running<false> {
  const float c;
  float m = kNegInf, z = 0.f, nmc = 0.f, delta = 0.f;
  int first = INT_MAX, cnt = 0;
  __device__ __forceinline__ explicit Running(float scale) : c(scale * kLog2e) {}
  __device__ __forceinline__ void raise(float gm, int first_vec, int n_vec) {
    const float nmc2 = -(gm * c);
    const float d2 = fmaf(gm, c, nmc2);
    z *= fast_exp2((m - gm) * c - delta + d2);   // m = -inf on first use: z stays 0
    m = gm; nmc = nmc2; delta = d2; first = first_vec; cnt = n_vec;
  }
  __device__ __forceinline__ float term(float v) const { return fast_exp2(fmaf(v, c, nmc)); }
  __device__ __forceinline__ void add(float a) { z += a; }
  __device__ __forceinline__ float sum_for(float M) const { return z * fast_exp2(-delta) * fast_exp2((m - M) * c); }
};

// e^t for -700 <= t <= 0 in float64: 2^n 2^f, n = rint(t log2 e), |f| <= 1/2, 2^f = 1 + f Q(f) with Q of degree 6 through the
// Chebyshev nodes of [-1/2, 1/2].  At most 1.1e-10 off relative, in proportion to |f|, so that e^0 is 1; NaN for a NaN.
__device__ __forceinline__ double exp_f64(double t) {
  constexpr double kLog2eD = 1.4426950408889634074, kRound = 0x1.8p52;       // adding kRound leaves n in the low bits
  constexpr double q[7] = {0.6931471805599453, 0.24022650922288757, 0.05550410883909618, 0.009618056678524627,
                           0.001333350238616314, 0.00015461444698573144, 1.529732376059561e-05};
  const double k = fma(t, kLog2eD, kRound);
  const double f = fma(t, kLog2eD, -(k - kRound));
  double p = q[6];
#pragma unroll
  for (int i = 5; i >= 0; --i) p = fma(p, f, q[i]);
  p = fma(p, f, 1.0);
  return __hiloint2double(__double2hiint(p) + (__double2loint(k) << 20), __double2loint(p));     // p 2^n
}

// Entropy sums of one thread (calibration), relative to its own running max m of the scaled logits x: S = sum e^t,
// U = sum t e^t, t = x - m, all in float64, as the entropy of short rows has them.  Bound by the vector ALU: 13 float64
// instructions an element, which take twice the slots of float32 ones here.  2112 rows of 126464: bf16 240 us, float32 265; the
// same pass over a float32 exponential with its argument corrected 165 and 205, but 1-3 % of its bf16 entropies were an ulp off
// where these are all the exact value rounded once; a float64 exponential of the library in a pass of its own 737 and 786.  Four
// chains side by side, and workgroups of 256 threads, measured alike.
struct EntropySums {
  double S = 0.0, U = 0.0, m = (double)kNegInf;
  __device__ __forceinline__ void raise(float x) {
    if (m > (double)kNegInf) {
      const double d = m - (double)x, f = exp(d);
      U = (U + d * S) * f;
      S *= f;
    }
    m = (double)x;
  }
  template <bool kGuard> __device__ __forceinline__ void add(float x) {
    const double t = (double)x - m;
    if (kGuard && (x == kNegInf || t < -700.0)) return;            // e^t < 1e-304; a NaN goes through to the sums
    const double e = exp_f64(t);
    S += e;
    U = fma(t, e, U);
  }
};

// kEnt: the row's entropy too, and conf from its sums (conf, tok may then be NULL).
template <typename T, int BLOCK, int U, bool kEnt, bool kFine>
__global__ void __launch_bounds__(BLOCK)
stage1_vec_kernel(const T *__restrict__ logits, int vocab, int mask_id, float scale,
                  RowFilter rf, float *__restrict__ conf, int32_t *__restrict__ tok, float *__restrict__ ent) {
  constexpr int N = Vec16<T>::N;
  constexpr bool kRaw = (sizeof(T) == 2);
  const int tid = threadIdx.x;
  int64_t out_row;
  if (!row_target(rf, blockIdx.x, &out_row)) {
    if (tid == 0 && out_row >= 0) {
      if (!kEnt || conf) { conf[out_row] = 0.f; tok[out_row] = -1; }
      if (kEnt) ent[out_row] = 0.f;
    }
    return;
  }
  constexpr bool kAnywhere = kEnt || kFine;      // the plain terms are for aligned rows
  // Rows of a vocabulary that is no multiple of N begin anywhere: up to N - 1 elements in front of the first whole vector and
  // behind the last one are taken by single threads.
  const T *__restrict__ row = logits + (int64_t)blockIdx.x * vocab;
  const int head = !kAnywhere ? 0 : (int)((16u - ((uint32_t)reinterpret_cast<uintptr_t>(row) & 15u)) & 15u) / (int)sizeof(T);
  const uint4 *__restrict__ p = reinterpret_cast<const uint4 *>(row + head);
  const int nvec = (vocab - head) / N;
  const int mask_vec = mask_id >= head ? (mask_id - head) / N : INT_MAX, mask_lane = mask_id >= head ? (mask_id - head) % N : 0;
  constexpr int kStride = BLOCK * U;

  // Main loop: groups of U vectors per thread, no bounds checks; then a one-vector-at-a-time
  // tail.  A thread visits vector indices in increasing order, so the group in which its
  // running max was first raised to its final value holds the lowest id attaining it.
  Running<kFine> run(kRaw ? scale : 1.0f);
  EntropySums es;
  auto single = [&](int id) {                    // element id alone
    if (id == mask_id) return;
    const float v = kRaw ? to_float(row[id]) : to_float(row[id]) * scale;
    if (v > run.m) { run.raise(v, id, 0); if (kEnt) es.raise(kRaw ? mul_rn(v, scale) : v); }
    if (kEnt) es.add<true>(kRaw ? mul_rn(v, scale) : v);
    else if (run.m > kNegInf) run.add(run.term(v));
  };
  if (kAnywhere && tid < head) single(tid);
  const int nfull = nvec / kStride;
  // The [MASK] column lies in exactly one group iteration of the whole block; only that
  // iteration pays for the per-vector check (the others would otherwise spend one predicated
  // select per element on it).
  const int it_mask = mask_vec / kStride;
  auto group = [&](int it, auto check_mask) {
    const int base = it * kStride + tid;
    uint4 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = load_stream(p + base + u * BLOCK);
    __builtin_amdgcn_sched_barrier(0);           // issue all U loads before touching any result
    float f[U][N];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec16<T>::unpack(w[u], f[u]);
      if (!kRaw) {
#pragma unroll
        for (int i = 0; i < N; ++i) f[u][i] *= scale;
      }
      if (decltype(check_mask)::value && base + u * BLOCK == mask_vec) {
#pragma unroll
        for (int i = 0; i < N; ++i) if (i == mask_lane) f[u][i] = kNegInf;
      }
    }
    float gm = kNegInf;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < N; ++i) gm = fmaxf(gm, f[u][i]);
    if (gm > run.m) { run.raise(gm, base, U); if (kEnt) es.raise(kRaw ? mul_rn(gm, scale) : gm); }
    if constexpr (kEnt) {
      float lo = f[0][0];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < N; ++i) lo = fminf(lo, f[u][i]);
      if ((double)(kRaw ? lo * scale : lo) - es.m > -700.0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < N; ++i) es.add<false>(kRaw ? mul_rn(f[u][i], scale) : f[u][i]);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < N; ++i) es.add<true>(kRaw ? mul_rn(f[u][i], scale) : f[u][i]);
      }
    } else if (!kFine || run.m > kNegInf) {
      float acc = 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < N; ++i) acc += run.term(f[u][i]);
      run.add(acc);
    }
  };
  const int split = it_mask < nfull ? it_mask : nfull;
  for (int it = 0; it < split; ++it) group(it, std::false_type{});
  if (it_mask < nfull) group(it_mask, std::true_type{});
  for (int it = split + 1; it < nfull; ++it) group(it, std::false_type{});
  for (int idx = nfull * kStride + tid; idx < nvec; idx += BLOCK) {
    float f[N];
    Vec16<T>::unpack(load_stream(p + idx), f);
    if (!kRaw) {
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] *= scale;
    }
    if (idx == mask_vec) {
#pragma unroll
      for (int i = 0; i < N; ++i) if (i == mask_lane) f[i] = kNegInf;
    }
    float gm = kNegInf;
#pragma unroll
    for (int i = 0; i < N; ++i) gm = fmaxf(gm, f[i]);
    if (gm > run.m) { run.raise(gm, idx, 1); if (kEnt) es.raise(kRaw ? mul_rn(gm, scale) : gm); }
    if constexpr (kEnt) {
#pragma unroll
      for (int i = 0; i < N; ++i) es.add<true>(kRaw ? mul_rn(f[i], scale) : f[i]);
    } else if (run.m > kNegInf) {                       // a vector holding only the mask column has no live value
#pragma unroll
      for (int i = 0; i < N; ++i) run.add(run.term(f[i]));
    }
  }

  if (kAnywhere && tid < vocab - head - nvec * N) single(head + nvec * N + tid);

  // ---- block reduction: max, then sum rescaled to the block max ----
  __shared__ float s_f[BLOCK / kWave];
  __shared__ int s_i[BLOCK / kWave];
  __shared__ double s_d[kEnt ? 2 * (BLOCK / kWave) : 1];
  const int lane = tid % kWave, wid = tid / kWave;
  float M = wave_max(run.m);
  if (lane == 0) s_f[wid] = M;
  __syncthreads();
  M = s_f[0];
#pragma unroll
  for (int i = 1; i < BLOCK / kWave; ++i) M = fmaxf(M, s_f[i]);
  __syncthreads();
  if constexpr (kEnt) {
    es.raise(kRaw ? mul_rn(M, scale) : M);              // a thread without a live value has empty sums
    wave_sum2(es.S, es.U);
    if (lane == 0) { s_d[2 * wid] = es.S; s_d[2 * wid + 1] = es.U; }
  } else {
    float zt = (run.m > kNegInf) ? run.sum_for(M) : 0.f;
    zt = wave_sum(zt);
    if (lane == 0) s_f[wid] = zt;
  }

  // ---- arg-max: lowest id attaining M.  Each thread whose own max equals M rescans the
  // (at most U) vectors of the iteration in which it first reached that max. ----
  int cand = INT_MAX;
  if (run.m == M && run.cnt == 0) cand = run.first;
  else if (run.m == M) {
    for (int u = 0; u < run.cnt && cand == INT_MAX; ++u) {
      const int idx = run.first + u * BLOCK;
      float f[N];
      Vec16<T>::unpack(p[idx], f);
#pragma unroll
      for (int i = N - 1; i >= 0; --i) {
        float v = kRaw ? f[i] : f[i] * scale;
        if (head + idx * N + i != mask_id && v == M) cand = head + idx * N + i;
      }
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o, kWave));
  if (lane == 0) s_i[wid] = cand;
  __syncthreads();
  if constexpr (kEnt) {
    double St = 0.0, Ut = 0.0;
#pragma unroll
    for (int i = 0; i < BLOCK / kWave; ++i) { St += s_d[2 * i]; Ut += s_d[2 * i + 1]; }
    const double H = log(St) - Ut / St;
    if (tid == 0) {
      ent[out_row] = (float)H;
      if (conf) {
        int best = INT_MAX;
#pragma unroll
        for (int i = 0; i < BLOCK / kWave; ++i) best = min(best, s_i[i]);
        conf[out_row] = (float)(1.0 / St);
        tok[out_row] = best;
      }
    }
  } else if (tid == 0) {
    float Z = 0.f;
    int best = INT_MAX;
#pragma unroll
    for (int i = 0; i < BLOCK / kWave; ++i) { Z += s_f[i]; best = min(best, s_i[i]); }
    conf[out_row] = 1.0f / Z;
    tok[out_row] = best;
  }
}

// Short rows (fewer than 256 vectors): one element per load.
template <typename T, int BLOCK>
__global__ void __launch_bounds__(BLOCK)
stage1_scalar_kernel(const T *__restrict__ logits, int vocab, int mask_id, float scale,
                     RowFilter rf, float *__restrict__ conf, int32_t *__restrict__ tok) {
  const int tid = threadIdx.x;
  int64_t out_row;
  if (!row_target(rf, blockIdx.x, &out_row)) {
    if (tid == 0 && out_row >= 0) { conf[out_row] = 0.f; tok[out_row] = -1; }
    return;
  }
  const T *__restrict__ p = logits + (int64_t)blockIdx.x * vocab;
  float m = kNegInf;
  int arg = INT_MAX;
  for (int w = tid; w < vocab; w += BLOCK) {
    if (w == mask_id) continue;
    const float x = scale * to_float(p[w]);
    if (x > m) { m = x; arg = w; }
  }
  __shared__ float s_f[BLOCK / kWave];
  __shared__ int s_i[BLOCK / kWave];
  const int lane = tid % kWave, wid = tid / kWave;
  float M = wave_max(m);
  if (lane == 0) s_f[wid] = M;
  __syncthreads();
  M = s_f[0];
  for (int i = 1; i < BLOCK / kWave; ++i) M = fmaxf(M, s_f[i]);
  __syncthreads();
  float z = 0.f;
  for (int w = tid; w < vocab; w += BLOCK) {
    if (w == mask_id) continue;
    z += fast_exp2((scale * to_float(p[w]) - M) * kLog2e);
  }
  z = wave_sum(z);
  int cand = (m == M) ? arg : INT_MAX;
  for (int o = kWave / 2; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o, kWave));
  if (lane == 0) { s_f[wid] = z; s_i[wid] = cand; }
  __syncthreads();
  if (tid == 0) {
    float Z = 0.f;
    int best = INT_MAX;
    for (int i = 0; i < BLOCK / kWave; ++i) { Z += s_f[i]; best = min(best, s_i[i]); }
    conf[out_row] = 1.0f / Z;
    tok[out_row] = best;
  }
}

}  // namespace

// ------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------
// Blocks of 1024 threads from 4096 vectors a row; below, a block that wide has one or two vectors a thread and its reductions
// outweigh them (120 MB of rows, 1024 -> 256 threads: bf16 2048 119 -> 52 us, 4096 84 -> 31, 8192 50 -> 25, 24576 27 -> 25;
// float32 4096 47 -> 21, 16384 alike).  Shorter rows than 256 vectors: one element per load.
template <typename T, bool kEnt>
static bool launch_vec(hipStream_t s, const T *logits, int64_t n_rows, int vocab, int mask_id, float scale, const RowFilter &rf,
                       float *conf, int32_t *tok, float *ent) {
  constexpr int N = Vec16<T>::N;
  const int nvec = vocab / N;
  const dim3 grid((unsigned)n_rows);
  constexpr int kWide = kEnt ? 512 : 1024;
  if constexpr (!kEnt) {
    if (nvec >= 4096 && vocab % N == 0 && (reinterpret_cast<uintptr_t>(logits) & 15u) == 0) {
      stage1_vec_kernel<T, kWide, 2, false, false><<<grid, kWide, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok, ent);
      return true;
    }
  }
  if (nvec >= 4096) stage1_vec_kernel<T, kWide, 2, kEnt, true><<<grid, kWide, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok, ent);
  else if (nvec >= 256) stage1_vec_kernel<T, 256, 2, kEnt, true><<<grid, 256, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok, ent);
  else return false;
  return true;
}

template <typename T>
static pvf_status launch_stage1_t(pvf_ctx *ctx, hipStream_t s, const T *logits, int64_t n_rows,
                                  int vocab, int mask_id, float scale, const RowFilter &rf,
                                  float *conf, int32_t *tok, float *ent) {
  if (ent ? launch_vec<T, true>(s, logits, n_rows, vocab, mask_id, scale, rf, conf, tok, ent)
          : launch_vec<T, false>(s, logits, n_rows, vocab, mask_id, scale, rf, conf, tok, nullptr)) {
    PVF_LAUNCH_CHECK(ctx, "stage1");
    return PVF_OK;
  }
  if (conf) stage1_scalar_kernel<T, 256><<<dim3((unsigned)n_rows), 256, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok);
  PVF_LAUNCH_CHECK(ctx, "stage1");
  return ent ? launch_entropy_short(ctx, s, logits, sizeof(T) == 2 ? PVF_BF16 : PVF_F32, n_rows, vocab, mask_id, scale, rf, ent) : PVF_OK;
}

pvf_status launch_stage1(pvf_ctx *ctx, hipStream_t s, const void *logits, int dtype,
                         int64_t n_rows, int vocab, int mask_id, float scale,
                         const RowFilter &rf, float *conf, int32_t *tok, float *ent) {
  if (n_rows == 0) return PVF_OK;
  PVF_REQUIRE(ctx, n_rows > 0 && n_rows < (1ll << 31), PVF_EINVAL, "stage1: n_rows=%lld out of range", (long long)n_rows);
  if (dtype == PVF_BF16)
    return launch_stage1_t<bf16_t>(ctx, s, static_cast<const bf16_t *>(logits), n_rows, vocab, mask_id, scale, rf, conf, tok, ent);
  return launch_stage1_t<float>(ctx, s, static_cast<const float *>(logits), n_rows, vocab, mask_id, scale, rf, conf, tok, ent);
}

}  // namespace pvf
