// Non-causal attention on the CDNA4 matrix cores (bf16, d_head = 128): every query of a
// canvas attends to all T positions of the same canvas, masked or not -- the denoiser sees
// the whole canvas at once (Sec. 2).  Flash-style: K / V tiles of 64 keys are staged in LDS,
// the softmax is kept online in registers and the T x T score matrix is never materialised.
//
// Layout choices
//   * one workgroup = 128 queries of one (canvas, head); 4 waves x 32 queries;
//   * scores are computed transposed, S^T = K Q^T (MFMA "A" = K rows, "B" = Q rows), so a lane
//     owns ONE query (column lane%32) and 32 of the tile's 64 keys in registers: the softmax
//     max / sum are register loops plus one exchange with lane^32;
//   * O^T = V^T P^T: the probabilities a lane just produced are already the "B" operand of
//     the second product (the contraction index is permuted identically on both operands), and
//     every O^T accumulator of a lane belongs to that lane's query, so rescaling is lane-local;
//   * V is read key-contiguous, from a [canvas, head, d_head, T rounded up to 64] copy written by the
//     rotary kernel or the QKV projection's epilogue; K and V^T tiles go global -> LDS directly, XOR-swizzled against bank conflicts,
//     double-buffered.
#include "common.h"

#include <type_traits>

namespace pvf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(1))) const void gptr_t;
typedef __attribute__((address_space(3))) void lptr_t;

constexpr int DH = 128, TQ = 128, TK = 64;
constexpr int kKTile = TK * DH * 2;          // 16 KB, [key][d] rows of 256 B
constexpr int kVTile = DH * TK * 2;          // 16 KB, [d][key] rows of 128 B
constexpr int kStage = kKTile + kVTile;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Eight values p >= 0 as p = x[0] + x[1] + x[2] in bf16, cut and not rounded: 8 bits each, so all 24 of a float32.  The two
// lower parts are at least 2^-126, which no sum shows, because a part of 0 would make a NaN of an infinite value.
__device__ __forceinline__ void split3(const float *p, bf16x8 *x) {
  typedef short short2v __attribute__((ext_vector_type(2)));
  constexpr short2v kTiny = {0x0080, 0x0080};
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = p[2 * e], b = p[2 * e + 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
      w[i][e] = __builtin_amdgcn_perm(ub, ua, 0x07060302);   // the upper halves
      if (i) w[i][e] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(short2v, w[i][e]), kTiny));
      a -= __uint_as_float(ua & 0xffff0000u);
      b -= __uint_as_float(ub & 0xffff0000u);
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) x[i] = __builtin_bit_cast(bf16x8, make_uint4(w[i][0], w[i][1], w[i][2], w[i][3]));
}

// Rows of the key-contiguous value buffers hold T rounded up to a whole tile of keys (vt_stride); what lies beyond T is
// never used.
//
// Window mode (K/V-cached rounds): the queries are the R window rows of a canvas (qkv holds only
// those rows); keys in the window [w0, w0 + n_valid) are read from there, every other key from the cache of the
// canvas' group (kc: rotated keys [T][d] row-major, vtc: values [head][d][vt_stride]).  Values are read in chunks of one
// 16-key group, so vt holds [seq][head][d][Rv] from the 16-key boundary at or below w0: where the window begins or
// ends inside a group, rope_vt_kernel has filled the rest of the group from the cache.
struct WinArgs {
  const bf16_t *kc, *vtc;
  int64_t group_stride;
  const int32_t *seq_slot, *row_pos;
  int32_t slots_per_group, R, Rv;
  // first position of a canvas' window; row_pos is -1 where the active block lies behind the canvas: an empty window at its end
  __device__ __forceinline__ int first(int seq, int T) const { return (int)min((uint32_t)row_pos[(int64_t)seq * R], (uint32_t)T); }
};

// SPLIT (window mode, launches that leave CUs idle): a workgroup takes 64 queries, which need only two of the four waves, and
// the loop over the key tiles is a chain of dependent steps of ~2 us each, so the waves work as two pairs: pair
// 0 takes the even key tiles, pair 1 the odd ones (two tiles are staged per step), and at the end pair 0 merges
// pair 1's running maximum, sum and O into its own.  Half as many steps for the same work.
//
// RAG: any canvas length and window alignment.  Keys beyond T in the last tile are read as key T - 1, get a score of
// -inf, and their value columns are cleared in LDS.  These shapes used to take a vector-ALU kernel that kept the
// probabilities in float32, so P goes into the second product as three bf16 parts (split3): all 24 bits of it, and an infinite
// value gives an infinity as it does there.  The even shapes keep the single bf16 P they always had.  Per layer, 32 heads:
// 3 canvases x 437 tokens 1196 us on that kernel, 34 with P in two parts (its last bits lost), 38 in three; four windows of 128
// rows over 715 tokens 1496, 25.6 and 27.6.
template <bool WIN, bool SPLIT, bool RAG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
attention_mfma_kernel(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ vt,
                      bf16_t *__restrict__ out, int T, int H, int vt_stride, WinArgs wa) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[(SPLIT ? 4 : 2) * kStage];
  static_assert(!SPLIT || WIN, "the key split exists in window mode only");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pair = SPLIT ? wave >> 1 : 0;                    // which half of the key tiles this wave takes
  const int qwave = SPLIT ? wave & 1 : wave;                 // which 32 queries
  const int fr = lane & 31, fh = lane >> 5;
  const int q0 = blockIdx.x * (SPLIT ? TQ / 2 : TQ), head = blockIdx.y, seq = blockIdx.z;
  const int d = H * DH;
  const int TQrows = WIN ? wa.R : T;                       // query rows per canvas in qkv / out
  const int64_t row0 = (int64_t)seq * TQrows;
  const bf16_t *qb = qkv + row0 * 3 * d + (int64_t)head * DH;
  const bf16_t *kb = qb + d;
  const bf16_t *vtb = vt + ((int64_t)seq * H + head) * DH * (WIN ? wa.Rv : vt_stride);
  int w0 = 0, w1 = 0;                                      // window = keys [w0, w1)
  int v0 = 0, v1 = 0;                                      // 16-key groups held by vt: keys [v0, v1)
  const bf16_t *kcb = nullptr, *vtcb = nullptr;
  if (WIN) {
    const int g = wa.seq_slot[seq] / wa.slots_per_group;
    w0 = wa.first(seq, T);
    w1 = w0 + min(wa.R, T - w0);
    v0 = w0 & ~15; v1 = (w1 + 15) & ~15;
    kcb = wa.kc + g * wa.group_stride + (int64_t)head * DH;
    vtcb = wa.vtc + g * wa.group_stride + (int64_t)head * DH * vt_stride;
  }

  // ---- Q fragments: "B" operand, column = query, k-chunk = 8 consecutive d ----
  const int qrow = min(q0 + qwave * 32 + fr, TQrows - 1);
  bf16x8 qf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8 *>(qb + (int64_t)qrow * 3 * d + ks * 16 + fh * 8);

  // ---- global -> LDS addressing (see file header) ----
  // K tile: slot s = i*256 + tid -> key s/16, position s%16, chunk = position ^ (key & 15)
  // V^T tile: slot s -> d-row s/8, position s%8, chunk = position ^ ((row >> 1) & 7)
  const bf16_t *k_src[4], *v_src[4];
  int k_key[4], k_col[4], v_row[4], v_key[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s = i * 256 + tid;
    const int key = s >> 4, kc = (s & 15) ^ (key & 15);
    k_src[i] = kb + (int64_t)key * 3 * d + kc * 8;
    k_key[i] = key; k_col[i] = kc * 8;
    const int vr = s >> 3, vc = (s & 7) ^ ((vr >> 1) & 7);
    v_src[i] = vtb + (int64_t)vr * vt_stride + vc * 8;
    v_row[i] = vr; v_key[i] = vc * 8;
  }
  auto issue_loads = [&](int kt, int slot) {                 // key tile kt -> LDS tile slot `slot`
    unsigned char *dst = lds + slot * kStage + wave * 1024;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16_t *ks, *vs;
      if (WIN) {
        int key = kt * TK + k_key[i];                      // canvas position of this K row
        if (RAG) key = min(key, T - 1);
        ks = (key >= w0 && key < w1) ? kb + (int64_t)(key - w0) * 3 * d + k_col[i]
                                     : kcb + (int64_t)key * d + k_col[i];
        const int vk = kt * TK + v_key[i];                 // first of the 8 keys of this V^T chunk
        vs = (vk >= v0 && vk < v1) ? vtb + (int64_t)v_row[i] * wa.Rv + (vk - v0)
                                   : vtcb + (int64_t)v_row[i] * vt_stride + vk;
      } else {
        ks = RAG ? kb + (int64_t)min(kt * TK + k_key[i], T - 1) * 3 * d + k_col[i] : k_src[i] + (int64_t)kt * TK * 3 * d;
        vs = v_src[i] + kt * TK;
      }
      __builtin_amdgcn_global_load_lds((gptr_t *)ks, (lptr_t *)(dst + i * 4096), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((gptr_t *)vs, (lptr_t *)(dst + kKTile + i * 4096), 16, 0, 0);
    }
  };

  floatx16 o[4];                      // O^T: [d tile][..], column = this lane's query
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[t][e] = 0.f;
  float m_run = -INFINITY;
  float l_rag = 0.f;                                         // RAG: running sum of P over this lane's keys
  floatx16 ol;                                               // ol[0] in lanes 0..31: running sum of P for query lane
#pragma unroll
  for (int e = 0; e < 16; ++e) ol[e] = 0.f;
  const floatx16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;                                               // "A" operand with row 0 = 1, rows 1..31 = 0
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)(fr == 0 ? 1.0f : 0.0f);
  const float c = kLog2e / sqrtf((float)DH);

  // per-lane LDS offsets of the operand reads; the buffer, the key sub-tile and the d tile are
  // compile-time offsets on top (the loop below is unrolled over the two buffers)
  int k_rd[8], v_rd[4];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) k_rd[ks] = fr * 256 + (((ks * 2 + fh) ^ (fr & 15)) << 4);
#pragma unroll
  for (int ks2 = 0; ks2 < 4; ++ks2) v_rd[ks2] = fr * 128 + (((2 * ks2 + fh) ^ ((fr >> 1) & 7)) << 4);

  const int nk = RAG ? (T + TK - 1) / TK : T / TK;
  // step = one key tile (SPLIT: two, one per pair); kBuf = which half of the double buffer holds it
  const int n_steps = SPLIT ? (nk + 1) / 2 : nk;
  auto stage_step = [&](int st, int buf) {
    if (SPLIT) {
      issue_loads(2 * st, 2 * buf);
      if (2 * st + 1 < nk) issue_loads(2 * st + 1, 2 * buf + 1);
    } else {
      issue_loads(st, buf);
    }
  };
  stage_step(0, 0);
  auto tile = [&](int st, auto buf_c) {
    constexpr int kBuf = decltype(buf_c)::value;
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    __syncthreads();
    if (st + 1 < n_steps) stage_step(st + 1, kBuf ^ 1);
    if (RAG && st + 1 == n_steps && T < nk * TK) {
      // the last tile: clear the value columns of keys >= T (4 consecutive keys per 8-byte piece)
      unsigned char *vlast = lds + (SPLIT ? 2 * kBuf + ((nk - 1) & 1) : kBuf) * kStage + kKTile;
      const int rem = T - (nk - 1) * TK;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int piece = i * 256 + tid;                     // 128 rows x 16 pieces
        const int row = piece >> 4, c8 = piece & 15;         // stored chunk c8 / 2, half c8 % 2
        const int valid = rem - (16 * (c8 >> 2) + 4 * ((c8 >> 1) & 1) + 8 * (c8 & 1));
        if (valid < 4) {
          uint64_t *p = reinterpret_cast<uint64_t *>(vlast + row * 128 + (((c8 >> 1) ^ ((row >> 1) & 7)) << 4) + (c8 & 1) * 8);
          *p = valid <= 0 ? 0 : *p & ((1ull << (16 * valid)) - 1);
        }
      }
      __syncthreads();
    }
    if (SPLIT && 2 * st + pair >= nk) return;    // an odd number of key tiles: pair 1 has none in the last step
    const unsigned char *ks_ = lds + (SPLIT ? 2 * kBuf + pair : kBuf) * kStage;
    const unsigned char *vs_ = ks_ + kKTile;

    // ---- S^T = K Q^T : 2 key sub-tiles x 8 k-steps ----
    floatx16 s[2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8 *>(ks_ + t * 32 * 256 + k_rd[ks]);   // key t*32 + fr
        // the first k-step starts from a constant zero accumulator: no registers to clear per tile
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], ks == 0 ? kZero16 : s[t], 0, 0, 0);
      }
    }
    if (RAG) {
      const int rem = T - (SPLIT ? 2 * st + pair : st) * TK;
      if (rem < TK) {                                        // accumulator e of sub-tile t: key 32 t + 8 (e / 4) + 4 fh + e % 4
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (t * 32 + 8 * (e >> 2) + 4 * fh + (e & 3) >= rem) s[t][e] = -INFINITY;
      }
    }
    // ---- online softmax for this lane's query ----
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[t][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // The running maximum moves only when the tile's maximum exceeds it by more than 8 in the exponent
    // (p then stays below 2^8, no overflow anywhere): the accumulators are rescaled in the first
    // tiles and almost never afterwards, instead of whenever one of the 32 queries sees a new maximum.
    const bool upd = (mx - m_run) * c > 8.0f;                // first tile: m_run = -inf
    const float m_new = upd ? mx : m_run;
    const float alpha = upd ? fast_exp2((m_run - m_new) * c) : 1.0f;   // first tile: exp2(-inf) = 0
    const float nmc = -m_new * c;
    bf16x8 pf[4];                                            // "B" operand of the 4 key k-steps
    float pr[RAG ? 4 : 1][8];                                // RAG: P, taken apart where it is multiplied
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u)                            // k-step u of sub-tile t: register groups 2u, 2u+1
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float p = fast_exp2(fmaf(s[t][8 * u + e], c, nmc));
          if constexpr (RAG) pr[2 * t + u][e] = p;
          else pf[2 * t + u][e] = (bf16_t)p;
        }
    m_run = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[t][e] *= alpha;
      if (RAG) l_rag *= alpha; else ol[0] *= alpha;
    }
    if (RAG) {
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) part[i] += pr[RAG ? i : 0][e];
      l_rag += (part[0] + part[1]) + (part[2] + part[3]);
    }
    // ---- O^T += V^T P^T : 4 d tiles x 4 key k-steps.  k slot (fh, e) of k-step ks2 is key
    //      16*ks2 + 4*fh + e (e < 4) or 16*ks2 + 8 + 4*fh + (e - 4): the order P came out in ----
#pragma unroll
    for (int ks2 = 0; ks2 < 4; ++ks2) {
      bf16x8 p3[3];
      if constexpr (RAG) split3(pr[ks2], p3);
      else p3[0] = pf[ks2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        // d row t*32 + fr; vt stores each group of 16 keys as {0-3, 8-11 | 4-7, 12-15}: chunk 2*ks2 + fh is this lane's 8 keys
        const bf16x8 vf = *reinterpret_cast<const bf16x8 *>(vs_ + t * 32 * 128 + v_rd[ks2]);
#pragma unroll
        for (int i = 0; i < (RAG ? 3 : 1); ++i) o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p3[i], o[t], 0, 0, 0);
      }
      // row sums of P on the matrix pipe (a "V^T" row of ones): the vector ALU is the busier unit here, but not with three parts
      if (!RAG) ol = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, p3[0], ol, 0, 0, 0);
    }
  };
  for (int st = 0; st + 1 < n_steps; st += 2) {
    tile(st, std::integral_constant<int, 0>{});
    tile(st + 1, std::integral_constant<int, 1>{});
  }
  if (n_steps & 1) tile(n_steps - 1, std::integral_constant<int, 0>{});
  // row 0 of that product: lane q % 32, register 0; RAG: the keys of this lane and of lane ^ 32
  float l_run = RAG ? l_rag + __shfl_xor(l_rag, 32, 64) : __shfl(ol[0], fr, 64);

  if (SPLIT) {
    // pair 1 hands (O, running maximum, running sum) of its key tiles to the wave of pair 0 with the same queries;
    // both are sums of 2^((s - m_pair) c) terms, so they meet after rescaling to the larger maximum
    __syncthreads();                                         // every wave is done with the tiles
    float *x = reinterpret_cast<float *>(lds) + qwave * 66 * 64 + lane;
    if (pair == 1) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) x[(t * 16 + e) * 64] = o[t][e];
      x[64 * 64] = m_run;
      x[65 * 64] = l_run;
    }
    __syncthreads();
    if (pair == 1) return;
    const float m1 = x[64 * 64], l1 = x[65 * 64];
    const float mm = fmaxf(m_run, m1);
    const float a0 = fast_exp2((m_run - mm) * c), a1 = fast_exp2((m1 - mm) * c);   // a pair without tiles: m = -inf, factor 0
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[t][e] = o[t][e] * a0 + x[(t * 16 + e) * 64] * a1;
    l_run = l_run * a0 + l1 * a1;
  }

  // ---- out[q][head*128 + d]: lane holds 4 consecutive d per accumulator group ----
  const int q = q0 + qwave * 32 + fr;
  if (q < TQrows) {
    const float inv = 1.0f / l_run;
    bf16_t *orow = out + (row0 + q) * d + (int64_t)head * DH;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bf16x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (bf16_t)(o[t][4 * i + j] * inv);
        *reinterpret_cast<bf16x4 *>(orow + t * 32 + 8 * i + 4 * fh) = v;
      }
  }
}

// Position of key t inside a key-contiguous vt row: bits 2 and 3 of t are swapped, so that every
// group of 16 keys is stored as {0-3, 8-11 | 4-7, 12-15}.  The 8 keys that one lane of the
// attention kernel feeds into a k-step of the P V product (the order in which the S^T accumulators
// hold them) are then one 16-byte chunk.
__device__ __forceinline__ int vt_pos(int t) { return (t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1); }

// Rotation of 8 pairs (i, i + 64) of a head: lo / hi hold elements i.. and i + 64.. in bf16, cs their (cos, sin).
__device__ __forceinline__ void rotate8(const uint4 &lo, const uint4 &hi, const float2 *cs, uint4 *ro, uint4 *rh) {
  const float4 *cs4 = reinterpret_cast<const float4 *>(cs);
  const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
  uint32_t ol[4], oh[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float4 c4 = cs4[e];                                // (cos, sin) of pairs 2e, 2e + 1
    const float a0 = __uint_as_float(lw[e] << 16), a1 = __uint_as_float(lw[e] & 0xffff0000u);
    const float b0 = __uint_as_float(hw[e] << 16), b1 = __uint_as_float(hw[e] & 0xffff0000u);
    const float2 r0 = rotate_pair(a0, b0, c4.x, c4.y), r1 = rotate_pair(a1, b1, c4.z, c4.w);
    const bf16_t l0 = (bf16_t)r0.x, l1 = (bf16_t)r1.x, h0 = (bf16_t)r0.y, h1 = (bf16_t)r1.y;
    ol[e] = (uint32_t)__builtin_bit_cast(uint16_t, l0) | ((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
    oh[e] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
  }
  *ro = make_uint4(ol[0], ol[1], ol[2], ol[3]);
  *rh = make_uint4(oh[0], oh[1], oh[2], oh[3]);
}

// Rotary embedding of q and k in place and the key-contiguous copy of v for whole canvases, one 256-thread workgroup per
// 64 canvas positions of one (canvas, head), with 16-byte accesses throughout:
// vt[canvas][head][d][vt_pos(t)] = v[canvas * T + t][head * 128 + d].
__global__ void __launch_bounds__(256)
rope_vt_kernel(bf16_t *__restrict__ qkv, bf16_t *__restrict__ vt, int T, int H, int vt_stride,
               const float2 *__restrict__ cos_sin) {
  __shared__ bf16_t tile[DH][64 + 2];
  const int tid = threadIdx.x, head = blockIdx.y, seq = blockIdx.z;
  const int d = H * DH, p0 = blockIdx.x * 64;
  bf16_t *base = qkv + ((int64_t)seq * T + p0) * 3 * d + (int64_t)head * DH;
  // rotate q and k: 64 rows x 2 tensors x 8 chunks of 8 pairs
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int idx = it * 256 + tid;
    const int ch = idx & 7, which = (idx >> 3) & 1, r = idx >> 4;
    if (p0 + r >= T) continue;
    bf16_t *p = base + (int64_t)r * 3 * d + which * d + ch * 8;
    const uint4 lo = *reinterpret_cast<const uint4 *>(p), hi = *reinterpret_cast<const uint4 *>(p + 64);
    uint4 ro, rh;
    rotate8(lo, hi, cos_sin + (int64_t)(p0 + r) * 64 + ch * 8, &ro, &rh);
    *reinterpret_cast<uint4 *>(p) = ro;
    *reinterpret_cast<uint4 *>(p + 64) = rh;
  }
  // transpose v through LDS: a thread reads 8 d of one row, then writes the 8 keys of one 16-byte vt chunk
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int idx = it * 256 + tid;
    const int rr = idx & 63, ch = idx >> 6;                  // consecutive lanes = consecutive rows: no bank conflicts
    uint4 v8 = make_uint4(0, 0, 0, 0);
    if (p0 + rr < T) v8 = *reinterpret_cast<const uint4 *>(base + (int64_t)rr * 3 * d + 2 * d + ch * 8);
    const uint32_t w[4] = {v8.x, v8.y, v8.z, v8.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[ch * 8 + 2 * e][rr] = __builtin_bit_cast(bf16_t, (uint16_t)(w[e] & 0xffffu));
      tile[ch * 8 + 2 * e + 1][rr] = __builtin_bit_cast(bf16_t, (uint16_t)(w[e] >> 16));
    }
  }
  __syncthreads();
  bf16_t *vb = vt + ((int64_t)seq * H + head) * DH * vt_stride + p0;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int idx = it * 256 + tid;
    const int g = idx & 7, dd = idx >> 3;                    // chunk g of vt row dd: keys 16 (g / 2) + 4 (g % 2) + {0-3, 8-11}
    const int k0 = 16 * (g >> 1) + 4 * (g & 1);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int kr = k0 + (e & 1) * 2 + (e >> 1) * 8;
      w[e] = (uint32_t)__builtin_bit_cast(uint16_t, tile[dd][kr]) | ((uint32_t)__builtin_bit_cast(uint16_t, tile[dd][kr + 1]) << 16);
    }
    *reinterpret_cast<uint4 *>(vb + (int64_t)dd * vt_stride + g * 8) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// The same for the window rows of a K/V-cached round, one workgroup per 16-key group of one (canvas, head): every thread has
// one chunk of each step.  Groups are counted from the 16-key boundary at or below the window's first row; row r of the
// window is position w0 + r (rows past the canvas end are padding, rotated like position T - 1).  vt row d, keys counted from
// that boundary; positions of a boundary group that lie outside the window come from the cache.
// PART: q, k and v come as the float32 partial sums of the split-K projection, part[split][row][3 d], added in split order and
// rounded to bf16 here; the v third of qkv is then not written (only the attention reads these rows).  Bound by latency:
// 64 rows, 8 splits: 9.4 us, where a reduction of its own and 64-row workgroups took 5.4 + 6.4.  All that a thread needs is asked for at
// once, behind one load (row_pos) for where the window lies; the registers that this takes (PART 128 instead of 56) cost nothing at any
// number of rows.  Windows that are and are not whole groups: 192 rows 8.8 -> 8.6 and 11.3 -> 10.9 us, 256 9.5 -> 9.2 and 13.3 -> 12.8, 320
// 10.6 -> 10.5 and 15.2 -> 15.1; behind whole sums 384 rows 6.7 -> 6.9 and 8.2 -> 7.8, 512 (are not) 9.4 -> 9.0, 640 11.0 -> 10.4.
template <bool PART>
__global__ void __launch_bounds__(256)
rope_vt_rows_kernel(bf16_t *__restrict__ qkv, const float *__restrict__ part, int splits, int M, bf16_t *__restrict__ vt, int T, int H,
                    int vt_stride, const float2 *__restrict__ cos_sin, WinArgs wa) {
  __shared__ bf16_t tile[DH][16 + 2];
  const int tid = threadIdx.x, head = blockIdx.y, seq = blockIdx.z;
  const int d = H * DH;
  const int g = wa.seq_slot[seq] / wa.slots_per_group;
  const int w0 = wa.first(seq, T), w1 = w0 + min(wa.R, T - w0);
  const int p0 = (w0 & ~15) + blockIdx.x * 16;               // first position of the group
  const int64_t row0 = (int64_t)seq * wa.R;
  // What a thread needs of the projection, in one go: 8 pairs of a rotated row (16 rows x 2 tensors x 8 chunks) and 8 d of a v row (16
  // rows x 16 chunks).  Threads without one read the window's first row.
  const int qk_ch = tid & 7, which = (tid >> 3) & 1, r = p0 - w0 + (tid >> 4), v_ch = tid >> 4, pos = p0 + (tid & 15);
  const bool qk_ok = r >= 0 && r < wa.R, v_ok = pos >= w0 && pos < w1;
  const int qk_col = which * d + head * DH + qk_ch * 8;
  const int64_t at[3] = {(row0 + (qk_ok ? r : 0)) * 3 * d + qk_col, (row0 + (qk_ok ? r : 0)) * 3 * d + qk_col + 64,
                         (row0 + (v_ok ? pos - w0 : 0)) * 3 * d + 2 * d + head * DH + v_ch * 8};
  uint4 in[3];
  if constexpr (!PART) {
#pragma unroll
    for (int i = 0; i < 3; ++i) in[i] = *reinterpret_cast<const uint4 *>(qkv + at[i]);
  } else {
    float a[3][8] = {};
    for (int z0 = 0; z0 < splits; z0 += 4) {                 // 4 splits in flight at a time
      float4 x[3][4], y[3][4];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 *p = reinterpret_cast<const float4 *>(part + (int64_t)min(z0 + j, splits - 1) * M * 3 * d + at[i]);
          x[i][j] = p[0]; y[i][j] = p[1];
        }
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (z0 + j < splits) {
            a[i][0] += x[i][j].x; a[i][1] += x[i][j].y; a[i][2] += x[i][j].z; a[i][3] += x[i][j].w;
            a[i][4] += y[i][j].x; a[i][5] += y[i][j].y; a[i][6] += y[i][j].z; a[i][7] += y[i][j].w;
          }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = (uint32_t)__builtin_bit_cast(uint16_t, (bf16_t)a[i][2 * e]) | ((uint32_t)__builtin_bit_cast(uint16_t, (bf16_t)a[i][2 * e + 1]) << 16);
      in[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
  if (qk_ok) {
    uint4 ro, rh;
    rotate8(in[0], in[1], cos_sin + (int64_t)min(w0 + r, T - 1) * 64 + qk_ch * 8, &ro, &rh);
    bf16_t *p = qkv + (row0 + r) * 3 * d + qk_col;
    *reinterpret_cast<uint4 *>(p) = ro;
    *reinterpret_cast<uint4 *>(p + 64) = rh;
  }
  {                                                          // v through LDS
    const int rr = tid & 15, ch = v_ch;
    uint4 v8 = make_uint4(0, 0, 0, 0);
    if (v_ok) {
      v8 = in[2];
    } else if (pos < T && pos < ((w1 + 15) & ~15)) {
      const bf16_t *vtcb = wa.vtc + g * wa.group_stride + ((int64_t)head * DH + ch * 8) * vt_stride + vt_pos(pos);
      uint16_t x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = __builtin_bit_cast(uint16_t, vtcb[(int64_t)e * vt_stride]);
      v8 = make_uint4(x[0] | ((uint32_t)x[1] << 16), x[2] | ((uint32_t)x[3] << 16), x[4] | ((uint32_t)x[5] << 16), x[6] | ((uint32_t)x[7] << 16));
    }
    const uint32_t w[4] = {v8.x, v8.y, v8.z, v8.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[ch * 8 + 2 * e][rr] = __builtin_bit_cast(bf16_t, (uint16_t)(w[e] & 0xffffu));
      tile[ch * 8 + 2 * e + 1][rr] = __builtin_bit_cast(bf16_t, (uint16_t)(w[e] >> 16));
    }
  }
  __syncthreads();
  const int h8 = tid & 1, dd = tid >> 1;                     // chunk h8 of vt row dd: keys 4 h8 + {0-3, 8-11} of the group
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int kr = 4 * h8 + (e & 1) * 2 + (e >> 1) * 8;
    w[e] = (uint32_t)__builtin_bit_cast(uint16_t, tile[dd][kr]) | ((uint32_t)__builtin_bit_cast(uint16_t, tile[dd][kr + 1]) << 16);
  }
  bf16_t *vb = vt + (((int64_t)seq * H + head) * DH + dd) * wa.Rv + blockIdx.x * 16 + h8 * 8;
  *reinterpret_cast<uint4 *>(vb) = make_uint4(w[0], w[1], w[2], w[3]);
}

}  // namespace

bool attention_mfma_supported(int dtype, int d_head) { return dtype == PVF_BF16 && d_head == DH; }

// Keys per row of the window rows' value buffer: whole key tiles from the 16-key boundary below the window.
int window_vt_stride(int R, int block_len, int prompt_len) {
  const int before = block_len % 16 == 0 && prompt_len % 16 == 0 ? 0 : 15;
  return (before + R + 63) / 64 * 64;
}

// 64-query workgroups whose wave pairs share the key tiles, where they do not outnumber the CUs (one per CU, by LDS): four
// windows of 128 rows over 715 keys 30.7 -> 25.6 us a layer (whole canvases gain nothing: 1 x 512 tokens 16.0 -> 17.2).  Up to
// 640 rows, like the splitting of K: above, a canvas's logits do not depend on what rides along.
static bool split_pays(int S, int rows, int n_heads) {
  return (int64_t)S * rows <= 640 && (int64_t)S * n_heads * ((rows + TQ / 2 - 1) / (TQ / 2)) <= 256;
}

// part: NULL, or the float32 partial sums of the split-K QKV projection [splits][S * R][3 d] that qkv_w is to be made from.  rotated:
// qkv_w and vt_w are what the attention reads.
pvf_status launch_window_attention_mfma(pvf_ctx *ctx, hipStream_t s, void *qkv_w, const float *part, int splits, void *vt_w, const void *kc,
                                        const void *vtc, int64_t group_stride, const int32_t *seq_slot, const int32_t *row_pos,
                                        const pvf_decode_cfg &cfg, int S, int n_heads, const float2 *cos_sin, void *out, bool rotated) {
  if (S == 0) return PVF_OK;
  const int T = cfg.prompt_len + cfg.gen_len, R = window_rows(cfg), vts = vt_keys(T);
  WinArgs wa;
  wa.kc = (const bf16_t *)kc; wa.vtc = (const bf16_t *)vtc; wa.group_stride = group_stride;
  wa.seq_slot = seq_slot; wa.row_pos = row_pos; wa.slots_per_group = 1 + cfg.K; wa.R = R;
  wa.Rv = window_vt_stride(R, cfg.block_len, cfg.prompt_len);
  // groups up to the end of the last key tile; what lies behind the window is not read
  const dim3 rgrid(wa.Rv / 16, n_heads, S);
  if (!rotated) {
    if (part) rope_vt_rows_kernel<true><<<rgrid, 256, 0, s>>>((bf16_t *)qkv_w, part, splits, S * R, (bf16_t *)vt_w, T, n_heads, vts, cos_sin, wa);
    else rope_vt_rows_kernel<false><<<rgrid, 256, 0, s>>>((bf16_t *)qkv_w, nullptr, 0, S * R, (bf16_t *)vt_w, T, n_heads, vts, cos_sin, wa);
    PVF_LAUNCH_CHECK(ctx, "rope_vt_rows");
  }
  // even: whole key tiles, whole 64-row blocks of window rows, windows that begin and end with a 16-key group
  const bool even = T % TK == 0 && R % 64 == 0 && cfg.block_len % 16 == 0 && cfg.prompt_len % 16 == 0;
  const bool split = R <= 64 || split_pays(S, R, n_heads);
  const int tq = split ? TQ / 2 : TQ;
  const dim3 grid((R + tq - 1) / tq, n_heads, S);
  const bf16_t *q = (const bf16_t *)qkv_w, *v = (const bf16_t *)vt_w;
  bf16_t *o = (bf16_t *)out;
  if (split && even) attention_mfma_kernel<true, true, false><<<grid, 256, 0, s>>>(q, v, o, T, n_heads, vts, wa);
  else if (split) attention_mfma_kernel<true, true, true><<<grid, 256, 0, s>>>(q, v, o, T, n_heads, vts, wa);
  else if (even) attention_mfma_kernel<true, false, false><<<grid, 256, 0, s>>>(q, v, o, T, n_heads, vts, wa);
  else attention_mfma_kernel<true, false, true><<<grid, 256, 0, s>>>(q, v, o, T, n_heads, vts, wa);
  PVF_LAUNCH_CHECK(ctx, "attention_window_mfma");
  return PVF_OK;
}

// qkv must already be rotated and vt [S][n_heads][128][vt_keys(T)] filled (launch_rope_vt, or the QKV projection's epilogue).
pvf_status launch_attention_mfma(pvf_ctx *ctx, hipStream_t s, const void *qkv, const void *vt,
                                 void *out, int S, int T, int n_heads) {
  if (S == 0) return PVF_OK;
  const dim3 grid((T + TQ - 1) / TQ, n_heads, S);
  if (T % TK == 0)
    attention_mfma_kernel<false, false, false><<<grid, 256, 0, s>>>((const bf16_t *)qkv, (const bf16_t *)vt, (bf16_t *)out, T, n_heads, T, WinArgs{});
  else
    attention_mfma_kernel<false, false, true><<<grid, 256, 0, s>>>((const bf16_t *)qkv, (const bf16_t *)vt, (bf16_t *)out, T, n_heads, vt_keys(T), WinArgs{});
  PVF_LAUNCH_CHECK(ctx, "attention_mfma");
  return PVF_OK;
}

pvf_status launch_rope_vt(pvf_ctx *ctx, hipStream_t s, void *qkv, void *vt, int S, int T,
                          int n_heads, const float2 *cos_sin) {
  if (S == 0) return PVF_OK;
  rope_vt_kernel<<<dim3(vt_keys(T) / 64, n_heads, S), 256, 0, s>>>((bf16_t *)qkv, (bf16_t *)vt, T, n_heads, vt_keys(T), cos_sin);
  PVF_LAUNCH_CHECK(ctx, "rope_vt");
  return PVF_OK;
}

}  // namespace pvf
