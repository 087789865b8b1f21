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
// U = sum t e^t, t = x - m, all in float64, as the entropy of short rows has them (float32 rows, and the bf16 rows that
// stage1_hist_kernel leaves).  Bound by the vector ALU: 13 float64
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
// kMarked: only rows whose entropy is kRereadRow.
constexpr uint32_t kRereadRow = 0x7fc0cafeu;     // a NaN that no computation makes

template <typename T, int BLOCK, int U, bool kEnt, bool kFine, bool kMarked = false>
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
  if (kMarked && __float_as_uint(ent[out_row]) != kRereadRow) return;
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

// Entropy, confidence and top-1 token of long bf16 rows (calibration) from a histogram: a bf16 row holds few distinct values,
// so the row is counted into LDS, 8192 counters for both signs of 32 exponents, and the float64 exponential is taken once
// per value that occurs instead of once per element -- the same terms as EntropySums adds, each weighted by its count.  The
// range ends four exponents above the largest one of a sample, 2048 elements at equal distances over the row; what lies outside
// goes to a list (1024 entries, added in one order afterwards) or, from -1.7e38 down, adds nothing beside any value above
// -1e38 (they are 700 apart at scales from 1e-35 on).  Rows of which this does not hold (more such elements, NaN, a maximum as low
// as that, a smaller scale) are left to stage1_vec_kernel in a launch behind this one (4.5 us where there are none), at once where
// the sample holds more than 1280 / vocab of them; so are rows of few values, told by equal elements of the sample: equal values
// of a wave wait for each other at their counter, and from a chance of 1 / 16 for two elements to be equal on an exponential for
// each is the quicker way (2112 rows of 126464: one value 170 against 970 us, 11 values 230 against 720, the last tenth of a row
// of one value 195 against 190).
// Bound by HBM and the LDS atomics together (2112 rows of 126464 of normal distribution 205-230 -> 108-115 us, 5 TB/s): per two
// elements 4 packed instructions for the counters' addresses, 3 for the maximum, 4 more, and 2 atomics.  Elements outside the range
// send their thread's 16 through a slower loop: 0.2 % of zeros 162 us, 0.5 % 210 (185-195 without counting); rows that are left at once
// take 5-15 us longer than without the attempt, and where the list just overflows, 40-60 % longer (1 % of zeros).
constexpr int kHistBlock = 512, kHistBins = 8192, kHistList = 1024;
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// y = bits - low of an element (16 bits): in range where bits 12..14 are 0; its counter is y ^ (y >> 3), 13 bits of it, which
// brings the sign down to bit 12 and permutes the other 12.
__device__ __forceinline__ float hist_value(int bin, uint32_t low) {
  uint32_t t = (uint32_t)bin & 0xfffu;
  t ^= t >> 3;
  t ^= t >> 6;
  return __uint_as_float((t + low + (((uint32_t)bin & 0x1000u) << 3)) << 16);
}

__global__ void __launch_bounds__(kHistBlock) __attribute__((amdgpu_waves_per_eu(8, 8)))
stage1_hist_kernel(const bf16_t *__restrict__ logits, int vocab, int mask_id, float scale, RowFilter rf, float *__restrict__ conf,
                   int32_t *__restrict__ tok, float *__restrict__ ent) {
  constexpr int N = 8, U = 2, kStride = kHistBlock * U;
  __shared__ uint32_t s_hist[kHistBins];
  __shared__ uint16_t s_list[kHistList];
  __shared__ int s_n, s_low, s_nan, s_ranges;            // list entries; whether an element below -1.7e38, a NaN occurred; ranges listed
  __shared__ int s_match, s_top, s_deep, s_out;          // of the sample: equal neighbours, largest exponent, 255 - the smallest, elements for the list
  __shared__ float s_f[kHistBlock / kWave];
  __shared__ int s_i[kHistBlock / kWave];
  __shared__ double s_d[2 * (kHistBlock / kWave)];
  const int tid = threadIdx.x, lane = tid % kWave, wid = tid / kWave;
  int64_t out_row;
  if (!row_target(rf, blockIdx.x, &out_row)) {
    if (tid == 0 && out_row >= 0) {
      if (conf) { conf[out_row] = 0.f; tok[out_row] = -1; }
      ent[out_row] = 0.f;
    }
    return;
  }
  const bf16_t *__restrict__ row = logits + (int64_t)blockIdx.x * vocab;
  const int head = (int)((16u - ((uint32_t)reinterpret_cast<uintptr_t>(row) & 15u)) & 15u) / 2;
  const uint4 *__restrict__ p = reinterpret_cast<const uint4 *>(row + head);
  const int nvec = (vocab - head) / N;
  const int mask_vec = mask_id >= head ? (mask_id - head) / N : INT_MAX, mask_lane = mask_id >= head ? (mask_id - head) % N : 0;
  // The sample: 32 pieces of 64 elements (whole lines) at equal distances over the row, nvec >= 3499, by the first waves.  Its lines
  // come from memory twice where many rows are under way (13824 rows of 71808: 0.6 % of the launch, 64 pieces 2.8 %).
  constexpr int kSample = kHistBlock / 2;
  const int sample_vec = tid / 8 * ((nvec - 8) / (kSample / 8 - 1)) + tid % 8;
  const uint4 sample = tid < kSample ? p[sample_vec] : make_uint4(0, 0, 0, 0);
  for (int i = tid; i < kHistBins / 4; i += kHistBlock) reinterpret_cast<uint4 *>(s_hist)[i] = make_uint4(0, 0, 0, 0);
  if (tid == 0) s_n = s_low = s_nan = s_ranges = s_match = s_top = s_deep = s_out = 0;
  __syncthreads();
  const uint32_t sw[4] = {sample.x, sample.y, sample.z, sample.w};
  if (tid < kSample) {                                   // whole waves
    int match = 0, top = 0, deep = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t o = __shfl(sw[i], (lane + 8) & (kWave - 1));     // of the next piece
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t a = h ? sw[i] >> 16 : sw[i] & 0xffffu, b = h ? o >> 16 : o & 0xffffu;
        match += __popcll(__ballot(a == b && a < 0xff00u));
        const int e = (int)(a >> 7) & 0xff;
        if (e < 254 && !(sample_vec == mask_vec && 2 * i + h == mask_lane)) top = max(top, e);
        if (a - 0xff00u > 0x80u) deep = max(deep, e < 254 ? 255 - e : 255);
      }
    }
    ushort2v td = {(unsigned short)top, (unsigned short)deep};
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
      td = __builtin_elementwise_max(td, __builtin_bit_cast(ushort2v, __shfl_xor(__builtin_bit_cast(uint32_t, td), o, kWave)));
    if (lane == 0) { atomicAdd(&s_match, match); atomicMax(&s_top, (int)td.x); atomicMax(&s_deep, (int)td.y); }
  }
  __syncthreads();
  const uint32_t low = (uint32_t)max((s_top ? s_top : 127) - 27, 0) << 7;      // bits of the smallest value counted
  if (255 - s_deep < (int)(low >> 7)) {                  // uniform: elements below the range, or beyond the ones that make it
    int out = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = i & 1 ? sw[i / 2] >> 16 : sw[i / 2] & 0xffffu;
      out += __popcll(__ballot(((a - low) & 0x7000u) != 0 && !(a >= 0xff00u && a <= 0xff80u)));
    }
    if (lane == 0 && out && tid < kSample) atomicAdd(&s_out, out);
    __syncthreads();
  }
  if (s_match > kSample * N / 16 || (int64_t)s_out * (vocab / (kSample * N)) > kHistList * 5 / 4) {      // uniform
    if (tid == 0) ent[out_row] = __uint_as_float(kRereadRow);
    return;
  }

  float m = kNegInf;
  int first = INT_MAX, cnt = 0;                          // vectors first, first + BLOCK, .. (cnt of them) raised m; cnt = 0: element first
  bool full = false;                                     // the list is: the row is read again, and this thread need not go on
  auto count_one = [&](uint32_t u) {                     // 16 bits of one element, whatever it is
    const uint32_t y = (u - low) & 0xffffu;
    if (!(y & 0x7000u)) { atomicAdd(&s_hist[(y ^ (y >> 3)) & 0x1fffu], 1u); return; }
    if (u == 0xff80u) return;                            // -inf
    if (u >= 0xff00u && u < 0xff80u) { s_low = 1; return; }
    if ((u & 0x7fffu) > 0x7f80u) { s_nan = 1; return; }
    if (s_n > kHistList) return;                         // full: the row is read again
    const int at = atomicAdd(&s_n, 1);
    if (at < kHistList) s_list[at] = (uint16_t)u;
  };
  auto single = [&](int id) {
    if (id == mask_id) return;
    const float v = to_float(row[id]);
    if (v > m) { m = v; first = id; cnt = 0; }
    count_one(__float_as_uint(v) >> 16);
  };
  // UV vectors of this thread from `base`, BLOCK apart; check_mask (uniform): the [MASK] column may lie in one.  (One instance of
  // the loop's body: with four of them their length showed in launches of few rows.)
  auto vectors = [&](int base, auto uv, bool check_mask) {
    constexpr int UV = decltype(uv)::value;
    uint4 w[UV];
#pragma unroll
    for (int u = 0; u < UV; ++u) w[u] = load_stream(p + base + u * kHistBlock);
    __builtin_amdgcn_sched_barrier(0);                   // issue all loads before touching any result
    uint32_t b[UV][4];
#pragma unroll
    for (int u = 0; u < UV; ++u) {
      b[u][0] = w[u].x; b[u][1] = w[u].y; b[u][2] = w[u].z; b[u][3] = w[u].w;
      if (check_mask && base + u * kHistBlock == mask_vec) {
#pragma unroll
        for (int i = 0; i < N; ++i)
          if (i == mask_lane) b[u][i / 2] = i & 1 ? (b[u][i / 2] & 0xffffu) | 0xff800000u : (b[u][i / 2] & 0xffff0000u) | 0xff80u;
      }
    }
    float gm = kNegInf;
    uint32_t bad = 0;
    const ushort2v low2 = {(unsigned short)low, (unsigned short)low};
#pragma unroll
    for (int u = 0; u < UV; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gm = fmaxf(fmaxf(gm, __uint_as_float(b[u][i] << 16)), __uint_as_float(b[u][i] & 0xffff0000u));
        const ushort2v y = __builtin_bit_cast(ushort2v, b[u][i]) - low2;
        bad |= __builtin_bit_cast(uint32_t, y);
      }
    if (gm > m) { m = gm; first = base; cnt = UV; }
    if ((bad & 0x70007000u) == 0) {
#pragma unroll
      for (int u = 0; u < UV; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          constexpr ushort2v k3 = {3, 3}, k2 = {2, 2};
          const ushort2v y = __builtin_bit_cast(ushort2v, b[u][i]) - low2;
          const ushort2v z = (y ^ (y >> k3)) << k2;      // byte address, bit 15 apart
          const uint32_t zz = __builtin_bit_cast(uint32_t, z);
          atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(s_hist) + (zz & 0x7fffu)), 1u);
          atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(s_hist) + ((zz >> 16) & 0x7fffu)), 1u);
        }
      return;
    }
    uint32_t every = b[0][0], some = b[0][0];
#pragma unroll
    for (int i = 1; i < UV * 4; ++i) { every &= b[i / 4][i % 4]; some |= b[i / 4][i % 4]; }
    if (every != 0xff80ff80u || some != 0xff80ff80u) {   // all -inf brings nothing
      uint32_t outside = 0;                              // bit 2 i + h: half h of word i
#pragma unroll
      for (int i = 0; i < UV * 4; ++i) {
        const uint32_t y = __builtin_bit_cast(uint32_t, __builtin_bit_cast(ushort2v, b[i / 4][i % 4]) - low2);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t z = h ? y >> 16 : y & 0xffffu, u = h ? b[i / 4][i % 4] >> 16 : b[i / 4][i % 4] & 0xffffu;
          if (!(z & 0x7000u)) atomicAdd(&s_hist[(z ^ (z >> 3)) & 0x1fffu], 1u);
          else if (u - 0xff00u > 0x80u) outside |= 1u << (2 * i + h);
          else if (u != 0xff80u) s_low = 1;              // -inf brings nothing
        }
      }
      while (outside) {
        const int k = __ffs(outside) - 1;
        outside &= outside - 1;
        uint32_t x = b[0][0];
#pragma unroll
        for (int q = 1; q < UV * 4; ++q) x = k / 2 == q ? b[q / 4][q % 4] : x;
        count_one(k & 1 ? x >> 16 : x & 0xffffu);
      }
      full = *(volatile int *)&s_n > kHistList;
    }
  };
  if (tid < head) single(tid);
  const int nfull = nvec / kStride, it_mask = mask_vec / kStride;
  const std::integral_constant<int, U> all{};
  for (int it = 0; it < nfull && !full; ++it) vectors(it * kStride + tid, all, it == it_mask);
  for (int idx = nfull * kStride + tid; idx < nvec; idx += kHistBlock) vectors(idx, std::integral_constant<int, 1>{}, true);
  if (tid < vocab - head - nvec * N) single(head + nvec * N + tid);
  float M = wave_max(m);
  if (lane == 0) s_f[wid] = M;
  __syncthreads();                                       // and every element is counted
  M = s_f[0];
#pragma unroll
  for (int i = 1; i < kHistBlock / kWave; ++i) M = fmaxf(M, s_f[i]);
  if (s_n > kHistList || s_nan || (s_low && !(M > -1e38f && scale >= 1e-35f))) {           // uniform
    if (tid == 0) ent[out_row] = __uint_as_float(kRereadRow);
    return;
  }
  // S = sum e^t, T = sum t e^t, t = x - max x, over the values that occur
  const double xm = (double)mul_rn(M, scale);
  double S = 0.0, T = 0.0;
  auto add = [&](float v, double n) {
    const float x = mul_rn(v, scale);
    const double t = (double)x - xm;
    if (x == kNegInf || t < -700.0) return;              // e^t < 1e-304; a NaN goes through to the sums
    const double e = exp_f64(t);
    S = fma(n, e, S);
    T = fma(n * t, e, T);
  };
  auto add_counts = [&](uint32_t from) {
    for (int i = tid; i < kHistBins; i += kHistBlock) {
      const uint32_t n = s_hist[i];
      if (n) add(hist_value(i, from), (double)n);
    }
  };
  add_counts(low);
  // The list is in the order of the atomics.  Up to 64 elements are sorted by their places in a wave; more are counted like the
  // others, 32 exponents after 32 (1.5-2 us for each such range that occurs): either way sums have one order.
  if (s_n <= kWave) {
    if (wid == 0) {
      const uint32_t v = lane < s_n ? s_list[lane] : 0u;
      int at = 0;
      for (int i = 0; i < s_n; ++i) {
        const uint32_t o = __shfl(v, i);
        at += o < v || (o == v && i < lane);
      }
      const uint32_t sorted = __builtin_amdgcn_ds_permute((lane < s_n ? at : lane) * 4, v);
      if (lane < s_n) add(__uint_as_float(sorted << 16), 1.0);
    }
  } else {
    for (int i = tid; i < s_n; i += kHistBlock) atomicOr(&s_ranges, 1 << (((s_list[i] - low) >> 12) & 7));
    __syncthreads();
    for (int r = 1; r < 8; ++r) {
      if (!(s_ranges >> r & 1)) continue;                // uniform
      const uint32_t from = low + (r << 12);
      for (int i = tid; i < kHistBins / 4; i += kHistBlock) reinterpret_cast<uint4 *>(s_hist)[i] = make_uint4(0, 0, 0, 0);
      __syncthreads();
      for (int i = tid; i < s_n; i += kHistBlock) {
        const uint32_t y = (s_list[i] - from) & 0xffffu;
        if (!(y & 0x7000u)) atomicAdd(&s_hist[(y ^ (y >> 3)) & 0x1fffu], 1u);
      }
      __syncthreads();
      add_counts(from);
      __syncthreads();
    }
  }
  wave_sum2(S, T);
  if (lane == 0) { s_d[2 * wid] = S; s_d[2 * wid + 1] = T; }
  // ---- arg-max: lowest id attaining M; a thread whose own maximum is M reads the vectors in which it first met it again ----
  int cand = INT_MAX;
  if (m == M && cnt == 0) cand = first;
  else if (m == M) {
    for (int u = 0; u < cnt && cand == INT_MAX; ++u) {
      const int idx = first + u * kHistBlock;
      float f[N];
      Vec16<bf16_t>::unpack(p[idx], f);
#pragma unroll
      for (int i = N - 1; i >= 0; --i)
        if (head + idx * N + i != mask_id && f[i] == M) cand = head + idx * N + i;
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o, kWave));
  if (lane == 0) s_i[wid] = cand;
  __syncthreads();
  if (tid == 0) {
    double St = 0.0, Tt = 0.0;
    int best = INT_MAX;
#pragma unroll
    for (int i = 0; i < kHistBlock / kWave; ++i) { St += s_d[2 * i]; Tt += s_d[2 * i + 1]; best = min(best, s_i[i]); }
    ent[out_row] = (float)(log(St) - Tt / St);
    if (conf) { conf[out_row] = (float)(1.0 / St); tok[out_row] = best; }
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
  // Counting pays from 28000 elements a row on, whatever the number of rows (which must not decide: a row's last bit would follow its
  // batch).  2112 rows: 16384 34.7 us either way, 20000 40 and 39, 32000 56 and 45; 64 rows, where the second launch shows: 20000 10.3
  // without and 11.7 with, 32000 15.1 and 13.2, 50257 14.0 and 14.2, 126464 28.5 and 21.4.
  if constexpr (kEnt && sizeof(T) == 2) {
    if (nvec >= 3500) {
      stage1_hist_kernel<<<grid, kHistBlock, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok, ent);
      stage1_vec_kernel<T, kWide, 2, true, true, true><<<grid, kWide, 0, s>>>(logits, vocab, mask_id, scale, rf, conf, tok, ent);
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
