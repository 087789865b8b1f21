// bf16 GEMM on the CDNA4 matrix cores:  C[M,N] = A[M,K] * W[N,K]^T, float32 accumulation,
// with the forward's fused epilogues (plain store, + residual, SwiGLU, and for the QKV projection
// the rotary embedding of q, k plus the key-contiguous copy of v).  These GEMMs are
// >90% of a PVF round's time (the batched forward over backbone + drafts, Sec. 4.1).
//
// Shape of the kernel
//   * workgroup tile BM x BN, WM x WN waves, each wave (BM/WM) x (BN/WN) as
//     v_mfma_f32_16x16x32_bf16 tiles (in a loop that also feeds LDS and direct loads this shape
//     sustains ~14% more than 32x32x16 at two waves per SIMD, although a loop of nothing but
//     MFMAs runs both at the same rate).  The shapes in use: 256 x 256 with 8 waves (2 x 4) for the
//     wide layers; 192 x 256, 128 x 256, 256 x 128, 160 x 256, 320 x 128, 192 x 128, 128 x 128 and (SwiGLU)
//     256 x 192, also with 8 waves, where they put (nearly) one tile on every CU; 64 x 64 and 64 x 128 with
//     4 waves and 128 x 64 with 8 for launches with few rows, which stream the weights and want many bytes on
//     the way (pick_config); launches of up to 640 rows may also split K over several workgroups per tile, as
//     nine shapes (splitk_plan); SwiGLU of 257-320 rows also takes 160 x 192 (swiglu_160x192_pays);
//   * both operands are K-contiguous in memory, so a 16-byte chunk is 8 consecutive k of one
//     row.  K advances in stages of BK = 64 (whole 128-byte lines per row: half the L2 requests
//     of 64-byte pieces) through a ring of LDS buffers; tiles go from
//     global memory straight into LDS (global_load_lds_dwordx4, no register staging) ahead of
//     the MFMAs; one raw s_barrier per stage, preceded by an explicit s_waitcnt vmcnt(n) that
//     lets the loads of later stages stay in flight (one per half stage where a wave tile is computed in
//     quadrants: 256 x 256, 192 x 256, 256 x 192).  The ring is as deep as the 160 KB of LDS
//     allow (two stages of the 256 x 256 tile, three of 160 x 256, five of 128 x 128): where a
//     stage lasts well under a microsecond the second stage of look-ahead is worth 10-15 %;
//   * an LDS row is 128 bytes (8 chunks); the chunk position is XOR-swizzled with
//     (row >> 1) & 7 so that the ds_read_b128 of an MFMA operand (16 consecutive rows, 4 chunk
//     positions) touches every bank once per 16 lanes.  The swizzle is applied by choosing
//     which global chunk a lane fetches, because the LDS slot of a direct load is fixed by the
//     lane id;
//   * the W tile is fed as the MFMA "A" operand and the activation tile as "B", so a lane ends
//     up with 4 consecutive output columns per accumulator group; the epilogue turns 32 rows at
//     a time around through LDS and stores whole 16-byte pieces of 128-byte lines;
//   * workgroup ids are remapped so that the 32 workgroups resident on one XCD (ids congruent
//     mod 8) cover a patch of 8 x 4 output tiles and share operand tiles through that XCD's L2.
#include "common.h"

#include <algorithm>
#include <climits>
#include <cstdlib>
#include <type_traits>

namespace pvf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));


typedef __attribute__((address_space(1))) const void gptr_t;
typedef __attribute__((address_space(3))) void lptr_t;

__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const bf16_t x = (bf16_t)a, y = (bf16_t)b;
  return (uint32_t)__builtin_bit_cast(uint16_t, x) | ((uint32_t)__builtin_bit_cast(uint16_t, y) << 16);
}

// s_waitcnt vmcnt(n) only (expcnt / lgkmcnt left at "no wait"); n is a 6-bit field split 4 + 2
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

// Whether a wave of WT columns holds the gate and the up column of an output: an even number of 16-column sub-tiles.
constexpr bool pairs_in_wave(int WT) { return WT / 16 % 2 == 0; }

constexpr bool is_rope(int epi) { return epi == kEpiQkvRope || epi == kEpiQkvRopeWin; }

// Row of W that feeds row r (0..BN-1) of the workgroup's W tile.
//  plain:   consecutive rows tile_n*BN + r.
//  SwiGLU:  the tile covers BN/2 output columns; the lower half of each wave's BN/WN tile rows is gate, the
//           upper half up for the same columns, so silu(g)*u pairs accumulators of one lane (16-row MFMA
//           sub-tiles c with NT16/2 + c).  Waves with an odd number of sub-tiles cannot: all gate columns of the tile come first.
//  QKV with rotary embedding (ff = 3 d): in the q and k thirds a wave's 64 tile rows are columns
//           [32g, 32g + 32) of a head followed by their rotation partners [64 + 32g, 64 + 32g + 32)
//           (g = wave % 2), so the pair (i, i + 64) meets in one lane (sub-tiles t and t + 2).
//  QKV of window rows (ff = 3 d, tiles of 64 columns): in the q and k thirds a tile is columns [32g, 32g + 32) of a head and
//           their partners (g = tile_n % 2), 16 and 16 a wave.
template <int EPI, int BN, int WN>
__device__ __forceinline__ int w_row(int r, int tile_n, int ff) {
  if (is_rope(EPI)) {
    if (tile_n * BN >= 2 * (ff / 3)) return tile_n * BN + r;           // v third: as it is
    const int wn = r >> 6, t = (r >> 4) & 3, e = r & 15;
    return tile_n * BN + (wn >> 1) * 128 + (t >> 1) * 64 + (wn & 1) * 32 + (t & 1) * 16 + e;
  }
  if (EPI == kEpiQkvWindow && tile_n * BN < 2 * (ff / 3))
    return (tile_n >> 1) * 128 + ((r >> 4) & 1) * 64 + (tile_n & 1) * 32 + (r >> 5) * 16 + (r & 15);
  if (EPI != kEpiSwiglu) return tile_n * BN + r;
  constexpr int WT = BN / WN;
  if (!pairs_in_wave(WT)) return (r < BN / 2 ? 0 : ff - BN / 2) + tile_n * (BN / 2) + r;
  const int wn = r / WT, e = r % (WT / 2);
  const int col = tile_n * (BN / 2) + wn * (WT / 2) + e;
  return r % WT >= WT / 2 ? ff + col : col;
}

// Quadrant schedule: LDS row r of an operand tile holds tile row half_row(r): first the lower halves of all wave tiles, then
// the upper ones, so that a half is a run of whole load instructions.
template <int BT, int WT> __device__ __forceinline__ int half_row(int r) {
  constexpr int kHalfTile = BT / 2, kHalfWave = BT / WT / 2;
  const int h = r / kHalfTile, rr = r % kHalfTile;
  return (rr / kHalfWave) * (2 * kHalfWave) + h * kHalfWave + rr % kHalfWave;
}

// workgroups per CU (by LDS) x waves per workgroup / 4 SIMDs
constexpr int waves_per_simd(int lds_bytes, int waves) { return (lds_bytes <= 80 * 1024 ? 2 : 1) * waves / 4; }

// kEpiQkvRope: the GEMM is the QKV projection of canvases of T tokens (d_head = 128, N = 3 * H * 128).
// Its epilogue rotates the q and k thirds (rotary embedding, pair (i, i + 64) of each head, angle
// of canvas position row % T from the cos_sin table [T][64]) before storing them, and writes the
// v third a second time key-contiguous, vt[canvas][head][d][t'] with bits 2 and 3 of t swapped in t'
// (each 16 keys stored as {0-3, 8-11 | 4-7, 12-15}), the layout the attention kernel reads its values in; a row of
// vt has Tv = vt_keys(T) entries.  Canvases of whole 16-key groups are written in 16-byte chunks, others key by key (the
// 64 keys of a column are then one or two runs of 2-byte stores).
struct RopeArgs {
  const float2 *cos_sin;
  bf16_t *vt;
  int32_t T, Tv, H;
  int32_t store_v;                                   // 0: the v third of C is not written (only vt)
  // window rows (kEpiQkvWindow, kEpiQkvRopeWin), windows of whole 16-key groups
  const int32_t *row_pos = nullptr;                  // canvas position of each row (negative: padding, rotated like position T - 1)
  int32_t R = 0;                                     // rows a canvas, a multiple of 16; Tv = keys of a row of vt
};

// kEpiPartial: the launch is split along K (blockIdx.y = split); every split stores its tile of float32
// partial sums to partial[split][M][N], which splitk_finalize_kernel adds up and finishes.
struct SplitK {
  float *partial;
  int32_t nk_per;                                    // k stages per split
  int32_t turn = 0;                                  // undivided launches: columns of tiles may start anywhere in K (host)
  int32_t ahead = 0, ahead8 = 0;                     // workgroups per XCD that only touch weights, for so many of 8 stages (touch_weights)
};

// Whether launches of a shape may have workgroups that touch weights (run): not the split ones, which fill the chip, nor 256 x 256.
constexpr bool touches(int epi, int bm, int bn) { return epi != kEpiPartial && bm * bn < 256 * 256; }

// A workgroup of a launch that leaves CUs idle in its last round: it reads a word of every 128-byte line of ahead8 of 8 stages of the
// weights of `tiles` tiles from `base` on, which its XCD runs in that round (every `ahead`-th column of tiles, from the p-th on), in the
// order in which their workgroups get there, so that those find part of the lines in L2.  What bounds them is not latency as such
// (deeper rings gain nothing; without MFMAs and LDS reads they take the same time) but that a CU has some 32 KB of loads on the way and
// takes them in order: activations that lie in L2 wait behind weights from HBM.  An idle CU has 32 KB of its own.
template <int EPI, int BN, int WN, int BK, int kThreads, bool kTurn>
__device__ __forceinline__ void touch_weights(const bf16_t *W, int p, int base, int tiles, int nk, int N_out, int K, int tiles_m, int tiles_n,
                                              int group_m, const SplitK &sk) {
  constexpr int kSide = kThreads / BN, kSlots = 4;           // columns or stages side by side, and loads of a thread on the way
  constexpr int kLines = 384;                                // lines to have on the way at least
  auto column = [&](int L) {                                 // columns of tiles in the order of their workgroups, band by band
    const int band = L / (group_m * tiles_n);
    return band * tiles_n + (L - band * (group_m * tiles_n)) / min(group_m, tiles_m - band * group_m);
  };
  const int first = column(base) + p, my_cols = (column(base + tiles - 1) - first + sk.ahead) / sk.ahead;      // at most kSide * kSlots (run)
  const int side = threadIdx.x / BN, row = threadIdx.x % BN;
  if (my_cols < 1 || side >= kSide) return;
  const int stages = max(1, min(kSide * kSlots / my_cols, (kLines + my_cols * BN - 1) / (my_cols * BN)));       // of an iteration
  const char *src[kSlots];
  int turn[kSlots], at[kSlots];
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const int u = side + j * kSide, tile_n = (first + u % my_cols * sk.ahead) % tiles_n;
    at[j] = u / my_cols;
    src[j] = at[j] < stages ? reinterpret_cast<const char *>(W) + (size_t)w_row<EPI, BN, WN>(row, tile_n, N_out) * (uint32_t)K * 2u : nullptr;
    turn[j] = kTurn ? (int)((uint32_t)(tile_n * nk) / (uint32_t)tiles_n) : 0;
  }
  constexpr int kFirst = 4;                                  // earlier stages are asked for by the time this workgroup runs
  uint32_t last[kSlots] = {};
  for (int i = 0; kFirst + i * 8 / sk.ahead8 < nk; i += stages) {
    uint32_t x[kSlots];
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      const int kt = kFirst + (i + at[j]) * 8 / sk.ahead8, kr = kt + turn[j] < nk ? kt + turn[j] : kt + turn[j] - nk;
      x[j] = src[j] && kt < nk ? *reinterpret_cast<const uint32_t *>(src[j] + kr * (BK * 2)) : 0;
    }
    asm volatile("" ::"v"(last[0]), "v"(last[1]), "v"(last[2]), "v"(last[3]));       // one iteration's words on the way while the next are asked for
#pragma unroll
    for (int j = 0; j < kSlots; ++j) last[j] = x[j];
  }
  asm volatile("" ::"v"(last[0]), "v"(last[1]), "v"(last[2]), "v"(last[3]));
}

template <int EPI, int BM, int BN, int BK, int kStages, int WM, int WN, bool kPairs, bool kHint, bool kTurn>
__global__ void __launch_bounds__(64 * WM * WN)
__attribute__((amdgpu_waves_per_eu(waves_per_simd(kStages * (BM + BN) * BK * 2, WM * WN),
                                   waves_per_simd(kStages * (BM + BN) * BK * 2, WM * WN))))
gemm_bf16_mfma_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                      bf16_t *__restrict__ C, const bf16_t *__restrict__ Res, int M, int N_out,
                      int K, int tiles_m, int tiles_n, int group_m, RopeArgs ra, SplitK sk, NormArgs na) {
  constexpr int kThreads = 64 * WM * WN;
  constexpr int MT = (BM / WM + 31) / 32;                  // 32-row passes of the epilogue (the last one may have 16 rows)
  constexpr int MT16 = BM / (16 * WM), NT16 = BN / (16 * WN);   // 16x16 MFMA tiles per wave in each direction
  constexpr int kATile = BM * BK * 2, kWTile = BN * BK * 2, kStage = kATile + kWTile;
  constexpr int CPR = BK / 8;                        // 16-byte chunks per LDS row
  constexpr int RPI = kThreads / CPR;                // tile rows covered by one load instruction of the block
  constexpr int kInstrBytes = kThreads * 16;         // LDS bytes filled by one load instruction of the block
  // A tile of 2.5 x RPI rows (160 x 256): the last A load instruction fills rows only from the lower half of the
  // block; the waves of the upper half repeat their previous load (same bytes to the same slot), so that every wave
  // has the same number of loads in flight and the same wait counts.
  constexpr bool kHalfA = BM % RPI != 0;
  constexpr int LA = (BM + RPI - 1) / RPI, LW = BN / RPI;        // direct loads per thread per stage
  constexpr int KS = BK / 32;                        // MFMA k-steps per stage
  constexpr int kRowBytes = BK * 2;
  // With a ring of only two stages (where the quadrant schedule cannot be taken) the refill of a slot is issued as soon as the slot is free (right
  // after the barrier in the last k-step of the stage that was read from it), all of it in that one
  // k-step: the loads of stage kt + 2 then have a whole stage to land.  Deeper rings spread the refill
  // of the slot freed one stage ago over the first k-steps of a stage.
  constexpr bool kLate = kStages == 2;
  // Rings of two stages whose wave tiles split into four equal quadrants run the quadrant schedule (quad_stage below).  It takes
  // the stages in pairs; an odd number of them (K % 128 == 64) has an instance of its own (kPairs = false) on the k-step
  // schedule.  With a tail for odd numbers beside the other one in one kernel the compiler spilled 100-400 registers.
  constexpr bool kQuad = kPairs && kLate && MT16 % 2 == 0 && NT16 % 2 == 0;
  // With whole load instructions per half of the W tile the W row of a lane is that of lane 0 plus a distance that is the
  // same for all loads, and one offset register does.
  constexpr bool kStepW = kQuad && (BN / 2) % RPI == 0;
  constexpr int kAhead = kLate ? kStages : kStages - 1;     // stages in flight after the prologue
  static_assert(BM % (RPI / 2) == 0 && (!kHalfA || LA >= 2) && BN % RPI == 0 && BK == 64 && BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "tile shape");
  // SwiGLU whose waves cannot pair gate and up turns the whole tile around through LDS.
  constexpr bool kTileStage = EPI == kEpiSwiglu && !pairs_in_wave(BN / WN);
  static_assert((!is_rope(EPI) && (EPI != kEpiSwiglu || kTileStage)) || BM % (32 * WM) == 0, "the rotary and SwiGLU epilogues take whole 32-row passes");
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: LDS targets become scalar arithmetic
  const int wm = wave / WN, wn = wave % WN;

  // ---- XCD-aware tile assignment ----
  const int total = tiles_m * tiles_n;
  const int chunk = (total + 7) >> 3;
  const int base = (blockIdx.x & 7) * chunk;
  if constexpr (touches(EPI, BM, BN)) if ((int)(blockIdx.x >> 3) >= chunk) {
    const int before = chunk & ~31, tiles = min(chunk, total - base) - before;           // in the rounds before the last, and in the last
    if (tiles > 0)
      touch_weights<EPI, BN, WN, BK, kThreads, kTurn>(W, (int)(blockIdx.x >> 3) - chunk, base + before, tiles, K / BK, N_out, K, tiles_m, tiles_n, group_m, sk);
    return;
  }
  const int L = base + (blockIdx.x >> 3);
  if (L >= total) return;
  const int band = L / (group_m * tiles_n);
  const int within = L - band * (group_m * tiles_n);
  const int band_rows = min(group_m, tiles_m - band * group_m);
  const int tile_n = within / band_rows;
  const int tile_m = band * group_m + (within - tile_n * band_rows);
  const int m0 = tile_m * BM;

  // ---- global -> LDS: thread tid fills 16-byte slot (i*kThreads + tid) of an operand tile:
  //      tile row i*RPI + tid/CPR, slot position tid%CPR, k-chunk position ^ swizzle(row) ----
  const int ld_row = tid / CPR;
  const int ld_chunk = (tid % CPR) ^ (CPR == 8 ? (ld_row >> 1) & 7 : (ld_row >> 2) & 3);
  // Per-lane byte offsets (32 bit) from the operand base; the k advance goes into the uniform
  // base pointer, so a load needs no per-lane address arithmetic.
  uint32_t a_off[LA], w_off[kStepW ? 1 : LW];
  uint32_t w_step[LW];                               // kStepW: uniform part of the W offsets
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int ar = kQuad ? half_row<BM, WM>(i * RPI + ld_row) : i * RPI + ld_row;
    const int am = min(m0 + ar, M - 1);                       // ragged last tile: re-read a valid row
    a_off[i] = ((uint32_t)am * (uint32_t)K + ld_chunk * 8) * 2u;
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    if (kStepW) {
      const int first = w_row<EPI, BN, WN>(half_row<BN, WN>(i * RPI), tile_n, N_out);
      w_step[i] = (uint32_t)first * (uint32_t)K * 2u;
      if (i == 0) w_off[0] = ((uint32_t)(w_row<EPI, BN, WN>(half_row<BN, WN>(ld_row), tile_n, N_out) - first) * (uint32_t)K + ld_chunk * 8) * 2u;
    } else {
      const int wr = kQuad ? half_row<BN, WN>(i * RPI + ld_row) : i * RPI + ld_row;
      w_off[i] = ((uint32_t)w_row<EPI, BN, WN>(wr, tile_n, N_out) * (uint32_t)K + ld_chunk * 8) * 2u;
    }
  }
  const char *Ab = reinterpret_cast<const char *>(A), *Wb = reinterpret_cast<const char *>(W);
  const uint32_t k_shift = EPI == kEpiPartial ? blockIdx.y * sk.nk_per * (BK * 2) : 0;     // this split's range of k
  Ab += k_shift;
  Wb += k_shift;
  constexpr int kLoadsPerStage = LA + LW;
  const int nk = EPI == kEpiPartial ? sk.nk_per : K / BK;
  // Split-K launches are bound by the weight stream, and with all workgroups at the same k their loads of a moment lie
  // K * 2 bytes apart, on few memory channels: each eighth of the tile columns starts an eighth of its k range further on and
  // wraps around.  An eighth of the columns is what one XCD has (up to the remainder where they are no multiple of 8), whose
  // workgroups share the activations in its L2.  By the column and not by the XCD itself: all tiles of a column, so all rows
  // of a launch, add their k in the same order, and equal rows stay equal.  Cached rounds 2.0 and 2.6 % faster.
  // So do launches of few rows that do not split K, every column of tiles from a place of its own: the 64-row tiles read the
  // activations from L2 wherever they are (64 rows: gate/up of 24576 weight rows 42.5 -> 35.5 us, QKV 24.5 -> 22.9).
  // And launches of 129-384 rows from K = 2048 on (gate/up of 2 x 12288, K = 4096: 192 rows 57.1 -> 53.0 us, 256 61.5 -> 58.4, 384 76.0
  // -> 72.5; 2 x 11520, K = 8192, 5-6 %; QKV of 384 rows 3 %; cached rounds of 192, 256 and 384 rows 1.3-2.3 %).  The other side: K = 1024
  // 2 % slower, 512 rows nothing in a round, 640 rows from 5 % quicker to 3 % slower.
  // An instance of its own: a division and a wrap per load in launches that do not turn cost 128 x 128 SwiGLU tiles 4-7 % at K <= 1024
  // (512 rows x 1408 columns, K = 512, 7.4 and 7.9 us).  tile_n nk < 2^19, as W is smaller than 4 GiB.
  const int turn = EPI == kEpiPartial ? nk / 8 * (tile_n * 8 / tiles_n) : kTurn ? (int)((uint32_t)(tile_n * nk) / (uint32_t)tiles_n) : 0;
  constexpr int kWAux = kHint ? 2 : 0;               // weights with the non-temporal hint (run)
  // The quadrant schedule loads through buffer descriptors: base + 32-bit lane offset + scalar offset, where the compiler
  // turns the global form into a 64-bit address per load and lane (16 registers that are not there).
  const int w_rows = EPI == kEpiSwiglu ? 2 * N_out : N_out;
#ifdef __HIP_DEVICE_COMPILE__                                // the descriptor type does not exist in the host pass
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void *)Ab, 0, (int)((uint32_t)M * (uint32_t)K * 2u - k_shift), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc((void *)Wb, 0, (int)((uint32_t)w_rows * (uint32_t)K * 2u - k_shift), 0x00020000);
#endif
  auto issue_one = [&](int kt, int i) {                      // load i (A loads first, then W) of stage kt
    unsigned char *dst = lds + (kt % kStages) * kStage + wave * 1024;
    const int kr = !(EPI == kEpiPartial || kTurn) || kt + turn < nk ? kt + turn : kt + turn - nk;
    if constexpr (kQuad) {
#ifdef __HIP_DEVICE_COMPILE__
      if (i < LA) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lptr_t *)(dst + i * kInstrBytes), 16, a_off[i], kr * (BK * 2), 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lptr_t *)(dst + kATile + (i - LA) * kInstrBytes), 16, w_off[kStepW ? 0 : i - LA], (kStepW ? w_step[i - LA] : 0u) + kr * (BK * 2), 0, kWAux);
#endif
      return;
    }
    const size_t koff = (size_t)kr * (BK * 2);
    if (i < LA) {
      const int ia = (kHalfA && i == LA - 1 && wave >= WM * WN / 2) ? i - 1 : i;      // uniform
      __builtin_amdgcn_global_load_lds((gptr_t *)(Ab + koff + a_off[ia]), (lptr_t *)(dst + ia * kInstrBytes), 16, 0, 0);
    } else
      __builtin_amdgcn_global_load_lds((gptr_t *)(Wb + koff + w_off[kStepW ? 0 : i - LA]), (lptr_t *)(dst + kATile + (i - LA) * kInstrBytes), 16, 0, kWAux);
  };

  // ---- LDS -> MFMA operands: lane reads row (base + lane%16), chunk (4*kk + lane/16) ----
  const int fr = lane & 15, fq = lane >> 4;
  const int swz = (fr >> 1) & 7;
  int frag_off[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) frag_off[kk] = fr * kRowBytes + (((kk * 4 + fq) ^ swz) << 4);
  const int a_base = wm * (BM / WM) * kRowBytes;             // byte offset of the wave's rows in the A tile
  const int w_base = kATile + wn * (BN / WN) * kRowBytes;

  floatx4 acc[NT16][MT16];                                   // [n sub-tile][m sub-tile]
#pragma unroll
  for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT16; ++mt)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[nt][mt][e] = 0.f;

  // Quadrant schedule: a stage's loads in the order in which their LDS rows are freed.  Group 1: the loads that lie in the
  // lower halves; group 2: the loads across the halves of an operand (192 rows) first, then the upper halves, W's before A's.
  constexpr int kLoA = (BM / 2) / RPI, kLoW = (BN / 2) / RPI;
  constexpr int kAcrossA = (BM / 2) % RPI != 0, kAcross = kAcrossA + ((BN / 2) % RPI != 0);
  constexpr int kG1 = kLoA + kLoW, kG2 = kLoadsPerStage - kG1;
  auto quad_load = [](int q) {                               // q-th load of a stage in that order
    if (q < kLoA) return q;
    if (q < kG1) return LA + q - kLoA;
    if (q < kG1 + kAcrossA) return kLoA;
    if (q < kG1 + kAcross) return LA + kLoW;
    const int u = q - kG1 - kAcross, nW = LW - kLoW - (kAcross - kAcrossA);        // upper rows
    return u < nW ? LW + LA - nW + u : LA - (kG2 - kAcross) + u;
  };
#pragma unroll
  for (int s = 0; s < kAhead; ++s)
    if (s < nk) {
#pragma unroll
      for (int i = 0; i < kLoadsPerStage; ++i) issue_one(s, kQuad ? quad_load(i) : i);
    }

  // Folded RMSNorm on the operand side: thread t < BM adds up the sums of squares of operand row m0 + t now,
  // while the first stages are in flight (8 loads at a time, slot order), and keeps 1 / rms for the epilogue.
  static_assert(BM <= kThreads, "one thread per tile row");
  float my_rnorm = 1.f;
  if ((EPI == kEpiSwiglu || is_rope(EPI)) && na.ss_in != nullptr && tid < BM) {
    const float *src = na.ss_in + min(m0 + tid, M - 1);
    float t = 0.f;
    for (int s0 = 0; s0 < na.n_slots_in; s0 += 8) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = s0 + j < na.n_slots_in ? src[(int64_t)(s0 + j) * na.ld] : 0.f;
#pragma unroll
      for (int j = 0; j < 8; j += 4) {
        if (na.group_in == 4) t += ((v[j] + v[j + 1]) + v[j + 2]) + v[j + 3];      // uniform
        else t = (((t + v[j]) + v[j + 1]) + v[j + 2]) + v[j + 3];
      }
    }
    my_rnorm = rsqrtf(t * na.inv_d + na.eps);
  }

  if constexpr (kQuad) {
    // A wave tile is computed in quadrants, each over the whole 64 k of a stage: (lower A, lower W), (lower, upper),
    // (upper, upper), (upper, lower).  An operand half is read from LDS one quadrant before it is first used, which frees its
    // rows early: one barrier per half stage hands half of a slot to the refill, so the loads of a stage are issued evenly
    // over a whole stage (all in the second half of one, they fill the CU's load path and the waves stand behind it) and
    // have 1-1.5 stages to land instead of 0.5-1.  Every element still adds its k in the same order.
    // Bound by the power budget and the load path (64 bytes a clock and CU).  Against the k-step schedule below, whole
    // forwards: 9 x 1280 rows 132.5 -> 125.5 ms, 5 x 512 29.3 -> 28.5, 80 x 1024 891 -> 870, 1 x 512 9.24 -> 8.88.
    constexpr int MH = MT16 / 2, NH = NT16 / 2, kPer = MH * NH * KS;
    constexpr int kBarrierAt = 4;                            // MFMAs of a half stage issued before its barrier
    constexpr int kSlots = 2 * kPer - kBarrierAt;            // MFMAs of a half stage behind it
    bf16x8 a0[MH][KS], a1[MH][KS], b[2][NH][KS];             // b[kt % 2]: the lower W half of stage kt
    const int a_off0 = wm * (BM / WM / 2) * kRowBytes, w_off0 = kATile + wn * (BN / WN / 2) * kRowBytes;
    auto rd_a = [&](const unsigned char *st, int half, int j) {          // j-th fragment in the order of use
      return *reinterpret_cast<const bf16x8 *>(st + a_off0 + half * (BM / 2) * kRowBytes + (j % MH) * 16 * kRowBytes + frag_off[j / MH]);
    };
    auto rd_w = [&](const unsigned char *st, int half, int j) {
      return *reinterpret_cast<const bf16x8 *>(st + w_off0 + half * (BN / 2) * kRowBytes + (j % NH) * 16 * kRowBytes + frag_off[j / NH]);
    };
    if (nk > 1) wait_vmcnt<kG2 - kAcross + kLoadsPerStage>(); else wait_vmcnt<kG2 - kAcross>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int j = 0; j < NH * KS; ++j) b[0][j % NH][j / NH] = rd_w(lds, 0, j);
#pragma unroll
    for (int j = 0; j < MH * KS; ++j) a0[j % MH][j / MH] = rd_a(lds, 0, j);
    auto quad_stage = [&](int kt, auto kind, auto parity) {   // kind: 0 = a stage that prefetches, 1 = the last but one, 2 = the last
      constexpr int P = decltype(parity)::value;
      constexpr bool kSteady = decltype(kind)::value == 0, more = decltype(kind)::value < 2;
      const unsigned char *stage = lds + P * kStage, *next = lds + (P ^ 1) * kStage;
#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const int mh = ph >> 1, nh = ph == 1 || ph == 2;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          const int kk = i / (MH * NH), mt = i % (MH * NH) / NH, nt = i % NH;
          if (i == kBarrierAt && (ph == 0 || (ph == 2 && more))) {
            // ph 0: all of stage kt has landed; ph 2: the lower halves of stage kt + 1 have (my parts of them)
            if (ph == 0) { if (more) wait_vmcnt<kLoadsPerStage>(); else wait_vmcnt<0>(); }
            else { if (kSteady) wait_vmcnt<kG2 - kAcross + kG1>(); else wait_vmcnt<kG2 - kAcross>(); }
            __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0): my reads of the rows that are refilled now are done
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
          }
          floatx4 &c = acc[nh * NH + nt][mh * MH + mt];
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[nh ^ P][nt][kk], mh ? a1[mt][kk] : a0[mt][kk], c, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < (ph == 0 || ph == 3 ? NH : MH) * KS; ++j) {
            constexpr int nA = MH * KS, nW = NH * KS;
            if (ph == 0 && i == kBarrierAt + j * (kPer - kBarrierAt - 2) / nW) b[P ^ 1][j % NH][j / NH] = rd_w(stage, 1, j);
            if (ph == 1 && i == j * (kPer - 2) / nA) a1[j % MH][j / MH] = rd_a(stage, 1, j);
            if (ph == 2 && more && i == kBarrierAt + j * (kPer - kBarrierAt) / nA) a0[j % MH][j / MH] = rd_a(next, 0, j);
            if (ph == 3 && more && i == j * (kPer - 4) / nW) b[P ^ 1][j % NH][j / NH] = rd_w(next, 0, j);
          }
          if (kSteady) {
            const int at = (ph & 1) * kPer + i - kBarrierAt;                  // MFMAs since the half's barrier
            constexpr int n1 = kG1, n2 = kG2;
#pragma unroll
            for (int q = 0; q < (ph < 2 ? n1 : n2); ++q)
              if (at == 1 + q * kSlots / (ph < 2 ? n1 : n2)) issue_one(kt + 2, quad_load(ph < 2 ? q : n1 + q));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    constexpr std::integral_constant<int, 0> k0{};
    constexpr std::integral_constant<int, 1> k1{};
    constexpr std::integral_constant<int, 2> k2{};
    for (int kt = 0; kt + 2 < nk; kt += 2) {
      quad_stage(kt, k0, k0);
      quad_stage(kt + 1, k0, k1);
    }
    quad_stage(nk - 2, k1, k0);                              // nk is even (run_cfg)
    quad_stage(nk - 1, k2, k1);
  } else {
  // Waits until at most n whole stages of this wave's direct loads are still in flight.
  auto wait_stages = [&](int n) {
    if (kStages >= 4 && n >= 2) wait_vmcnt<2 * kLoadsPerStage>();
    else if ((kStages >= 3 || kLate) && n >= 1) wait_vmcnt<kLoadsPerStage>();
    else wait_vmcnt<0>();
  };
  // Operand fragments of a k-step (32 k).  The A fragments and the W fragment of the last pass
  // are double-buffered in registers; the other W fragments are single register sets that are
  // re-read for the next k-step right after the pass that used them.
  static_assert(KS % 2 == 0, "the register double buffer alternates with the k-step inside a stage");
  bf16x8 af[2][MT16], wf[NT16 - 1], wl[2];
  auto read_a = [&](const unsigned char *stage, int kk, int buf, int mt) {
    af[buf][mt] = *reinterpret_cast<const bf16x8 *>(stage + a_base + mt * 16 * kRowBytes + frag_off[kk]);
  };
  auto read_w = [&](const unsigned char *stage, int kk, int buf, int nt) {
    const bf16x8 v = *reinterpret_cast<const bf16x8 *>(stage + w_base + nt * 16 * kRowBytes + frag_off[kk]);
    if (nt == NT16 - 1) wl[buf] = v; else wf[nt] = v;
  };

  // Software pipeline over k-steps, written out in issue order and pinned with sched_barrier
  // after every MFMA: a wave issues in order, so whatever stands between two MFMAs must fit into
  // the cycles the first one keeps the matrix pipe busy.  A k-step runs its MFMAs n sub-tile by
  // n sub-tile (a "pass" = one W fragment against all A fragments).  The LDS reads for the NEXT
  // k-step follow single MFMAs and are all issued before the last pass starts, so a k-step never
  // begins by waiting for LDS.  The direct loads that fall to a k-step follow one MFMA each.
  // In the LAST k-step of stage kt the wave, kBarrierAt MFMAs in, waits for its own direct loads
  // of stage kt+1 and passes the block's one barrier per stage (its LDS reads of stage kt were
  // issued a pass or more ago); the fragments it reads after that are the first ones of stage kt+1.
  // A steady stage (one that still prefetches) has compile-time wait counts and no branches.
  constexpr int kMfmaPerStep = MT16 * NT16;
  constexpr int kVmPerStep = KS > 1 ? (kLoadsPerStage + KS - 2) / (KS - 1) : kLoadsPerStage;
  constexpr int kLateStride = (MT16 * NT16 - 4) / (LA + LW) >= 2 ? 2 : 1;   // every second MFMA where the k-step is long enough
  constexpr int kBarrierAt = MT16 - 1 < 4 ? MT16 - 1 : 4;   // MFMAs of the last k-step issued before the barrier
  // the A reads are spread over MFMAs (kBarrierAt, kReadEnd): up to the start of the last pass
  constexpr int kReadEnd = (NT16 - 1) * MT16 > kBarrierAt + 2 ? (NT16 - 1) * MT16 : kBarrierAt + 2;
  static_assert(!kLate || kLoadsPerStage * kLateStride <= kMfmaPerStep - kBarrierAt + kLateStride - 1, "the refill loads fit into the last k-step");
  static_assert(kReadEnd <= kMfmaPerStep, "the A reads fit into the k-step");
  wait_stages(min(kAhead - 1, nk - 1));
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int nt = 0; nt < NT16; ++nt) read_w(lds, 0, 0, nt);
#pragma unroll
  for (int mt = 0; mt < MT16; ++mt) read_a(lds, 0, 0, mt);
  auto run_stage = [&](int kt, auto steady) {
    constexpr bool kSteady = decltype(steady)::value;
    const unsigned char *stage = lds + (kt % kStages) * kStage;
    const unsigned char *next = lds + ((kt + 1) % kStages) * kStage;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
      const bool last = kk + 1 == KS;
      const bool more = !last || kSteady || kt + 1 < nk;     // is there a next k-step to read for
      const unsigned char *src = last ? next : stage;
      const int skk = last ? 0 : kk + 1;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kMfmaPerStep; ++i) {
        const int nt = i / MT16, mt = i % MT16;
        if (last && more && i == kBarrierAt) {
          if (kSteady) wait_vmcnt<(kStages - 2) * kLoadsPerStage>();   // stage kt+1 has landed (my part of it)
          else wait_stages(min(kStages - 2, nk - 2 - kt));
          __builtin_amdgcn_s_waitcnt(0xc07f);                // lgkmcnt(0): my reads of stage kt are done
          // Raw barrier (no fence): every wave has waited for its own direct loads and LDS reads.
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nt == NT16 - 1 ? wl[cur] : wf[nt], af[cur][mt], acc[nt][mt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
          if (i == kBarrierAt) read_w(src, skk, nxt, NT16 - 1);
#pragma unroll
          for (int m2 = 0; m2 < MT16; ++m2)
            if (i == kBarrierAt + 1 + (m2 * (kReadEnd - kBarrierAt - 1)) / MT16) read_a(src, skk, nxt, m2);
          if (mt == MT16 - 1 && nt < NT16 - 1) read_w(src, skk, nxt, nt);
        }
        if (!kLate && kSteady && !last) {
#pragma unroll
          for (int q = 0; q < kVmPerStep; ++q)
            if ((q * kMfmaPerStep) / kVmPerStep == i && kk * kVmPerStep + q < kLoadsPerStage)
              issue_one(kt + kStages - 1, kk * kVmPerStep + q);
        }
        // slot kt % kStages was freed by the barrier above: one refill load after every kLateStride-th MFMA
        if (kLate && kSteady && last && i >= kBarrierAt && (i - kBarrierAt) % kLateStride == 0 &&
            (i - kBarrierAt) / kLateStride < kLoadsPerStage)
          issue_one(kt + kStages, (i - kBarrierAt) / kLateStride);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  const int n_loading = nk - kAhead;                         // stages that still have a stage to prefetch
  int kt = 0;
  for (; kt < n_loading; ++kt) run_stage(kt, std::true_type{});
  for (; kt < nk; ++kt) run_stage(kt, std::false_type{});
  }

  if constexpr (EPI == kEpiQkvWindow) {
    // Window rows of K/V-cached rounds whose windows are whole 16-key groups: q and k rotated, v key-contiguous, each from the wave's
    // own piece of the free ring, rounded as the rotary pass would find and leave them.  Saves that pass (4.9 us a layer at 64 rows) and
    // its launch: cached rounds of 64 rows 4.10 -> 4.04 ms, 128 rows 4.84 -> 4.63 (four canvases), 4.80 -> 4.73 (one).
    static_assert(BN == 64 && WN == 2 && MT16 == 2 && NT16 == 2, "waves of 32 x 32");
    constexpr int kRow = 32 * 2 + 16;
    const int d = N_out / 3, third = tile_n * BN / d;
    unsigned char *my = lds + wave * 32 * kRow;
    float4 cs[2][2];
    if (third < 2)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int pos = ra.row_pos[min(m0 + wm * 32 + h * 16 + fr, M - 1)];
        const float4 *p = reinterpret_cast<const float4 *>(ra.cos_sin + (int64_t)(pos < 0 ? ra.T - 1 : pos) * 64 + (tile_n & 1) * 32 + wn * 16 + 4 * fq);
        cs[h][0] = p[0]; cs[h][1] = p[1];
      }
    __syncthreads();                                                 // every wave is done with the ring
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t lo[2], up[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        lo[e] = pack_bf16x2(acc[0][h][2 * e], acc[0][h][2 * e + 1]);
        up[e] = pack_bf16x2(acc[1][h][2 * e], acc[1][h][2 * e + 1]);
        if (third < 2) {
          const float2 r0 = rotate_pair(__uint_as_float(lo[e] << 16), __uint_as_float(up[e] << 16), cs[h][e].x, cs[h][e].y);
          const float2 r1 = rotate_pair(__uint_as_float(lo[e] & 0xffff0000u), __uint_as_float(up[e] & 0xffff0000u), cs[h][e].z, cs[h][e].w);
          lo[e] = pack_bf16x2(r0.x, r1.x);
          up[e] = pack_bf16x2(r0.y, r1.y);
        }
      }
      unsigned char *row = my + (h * 16 + fr) * kRow + 4 * fq * 2;
      *reinterpret_cast<uint2 *>(row) = make_uint2(lo[0], lo[1]);
      *reinterpret_cast<uint2 *>(row + 32) = make_uint2(up[0], up[1]);
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int piece = it * 64 + lane;
      if (third < 2) {                                               // row piece / 4: 16 columns below, 16 above
        const int r = piece >> 2, c = piece & 3, m = m0 + wm * 32 + r;
        if (m < M) *reinterpret_cast<uint4 *>(C + (int64_t)m * N_out + (tile_n >> 1) * 128 + (c >> 1) * 64 + (tile_n & 1) * 32 + wn * 16 + (c & 1) * 8) =
                       *reinterpret_cast<const uint4 *>(my + r * kRow + c * 16);
      } else {                                                       // column piece / 4: chunk piece % 4 of its 32 keys
        const int c = piece >> 2, kg = piece & 3, m = m0 + wm * 32 + 16 * (kg >> 1), col = tile_n * BN - 2 * d + wn * 32 + c;
        const unsigned char *src = my + (16 * (kg >> 1) + 4 * (kg & 1)) * kRow + c * 2;
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int kr = (e & 1) * 2 + (e >> 1) * 8;
          w[e] = *reinterpret_cast<const uint16_t *>(src + kr * kRow) | ((uint32_t)*reinterpret_cast<const uint16_t *>(src + (kr + 1) * kRow) << 16);
        }
        if (m < M)
          *reinterpret_cast<uint4 *>(ra.vt + (((int64_t)(m / ra.R) * ra.H + (col >> 7)) * 128 + (col & 127)) * ra.Tv + m % ra.R + (kg & 1) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
    return;
  }
  if constexpr (kTileStage) {
    // 160 x 192: the sums as float32 rows in the free ring (16 bytes of padding: rows start 4 banks apart), then gate and up from
    // there.  Against float32 partial sums through memory and a launch that pairs them: 320 rows of gate/up, 2 x 12288 columns, K =
    // 4096, 68.3 -> 58.3 us.
    constexpr int kRow = BN * 4 + 16, kCols8 = BN / 16;       // 8-column pieces of an output row
    static_assert(BM * kRow <= kStages * kStage && BN % 16 == 0, "the tile exceeds the LDS ring");
    __syncthreads();                                                 // every wave is done with the ring
#pragma unroll
    for (int mt = 0; mt < MT16; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt)
        *reinterpret_cast<floatx4 *>(lds + (wm * (BM / WM) + mt * 16 + fr) * kRow + (wn * (BN / WN) + nt * 16 + 4 * fq) * 4) = acc[nt][mt];
    __syncthreads();
    for (int i = tid; i < BM * kCols8; i += kThreads) {
      const int r = i / kCols8, c = i % kCols8 * 8, m = m0 + r;
      if (m >= M) break;                                             // rows only grow
      const floatx4 *g = reinterpret_cast<const floatx4 *>(lds + r * kRow + c * 4), *u = reinterpret_cast<const floatx4 *>(lds + r * kRow + (BN / 2 + c) * 4);
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = silu_f(g[e >> 2][e & 3]) * u[e >> 2][e & 3];
      *reinterpret_cast<uint4 *>(C + (int64_t)m * N_out + tile_n * (BN / 2) + c) =
          make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
    return;
  }
  // ---- epilogue ----
  // A lane holds, for sub-tile (nt, mt), the 4 consecutive columns nt*16 + 4*(lane/16) + {0..3}
  // of row mt*16 + lane%16, so a direct store would write 8-byte pieces.  Instead each wave turns 32 rows at a time
  // around through its own piece of the (now free) LDS ring and stores 16 bytes per lane with
  // consecutive lanes along a row (whole 128-byte lines).  Staging is bf16 except for the
  // residual epilogue, which stages float32 so that acc + residual is rounded once.
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int OC = (EPI == kEpiSwiglu) ? WTN / 2 : WTN;            // output columns of this wave
  constexpr bool kStageF32 = EPI == kEpiResidual || EPI == kEpiPartial;
  constexpr int kElem = kStageF32 ? 4 : 2;
  constexpr int kStride = OC * kElem + 16;                           // padded row of the staging area
  constexpr int LPR = OC / 8;                                        // lanes per output row (8 columns each)
  constexpr bool kWholeRows = 64 % LPR == 0;                         // a store instruction covers whole rows (not with 48 columns)
  constexpr int kRowsPerInstr = 64 / LPR;                            // kWholeRows only
  static_assert(WM * WN * 32 * kStride <= kStages * kStage, "staging area exceeds the LDS ring");
  const int out_col0 = (EPI == kEpiSwiglu ? tile_n * (BN / 2) : tile_n * BN) + wn * OC;
  const int rd_row = lane / LPR, rd_col0 = (lane % LPR) * 8;
  // row (of the 32 of a pass) and columns that this lane stores with instruction j
  auto st_row = [&](int j) { return kWholeRows ? j * kRowsPerInstr + rd_row : (j * 64 + lane) / LPR; };
  auto st_col = [&](int j) { return kWholeRows ? rd_col0 : (j * 64 + lane) % LPR * 8; };
  static_assert(kTileStage || (32 * LPR % 64 == 0 && (kWholeRows || WTM % 32 == 0 || EPI == kEpiPartial)), "whole store instructions per pass");
  // The residual rows of the whole wave tile are requested at once, before the staging starts:
  // fetched 32 rows at a time where they are added, each piece cost a full memory latency.
  constexpr int kRowIters = 32 * LPR / 64;
  static_assert(kWholeRows || EPI == kEpiPartial || EPI == kEpiSwiglu || EPI == kEpiQkvWindow, "the other epilogues store whole rows per instruction");
  uint4 rs[EPI == kEpiResidual ? MT : 1][kRowIters];
  if (EPI == kEpiResidual) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < kRowIters; ++j) {
        if (mt * 32 + j * kRowsPerInstr >= WTM) continue;            // beyond a last pass of 16 rows
        const int m = m0 + wm * WTM + mt * 32 + j * kRowsPerInstr + rd_row;
        rs[mt][j] = make_uint4(0, 0, 0, 0);
        if (m < M) rs[mt][j] = *reinterpret_cast<const uint4 *>(Res + (int64_t)m * N_out + out_col0 + rd_col0);
      }
  }
  __syncthreads();                                                   // every wave is done with the ring
  // Folded RMSNorm: kNormOff bytes into the (free) ring lie above every staging area.  A reading projection
  // puts 1 / rms of its BM operand rows there; a writing one collects the row sums of squares of its output.
  // (The small tiles of the few-row launches have no room for it and never take part.)
  constexpr int kNormOff = 80 * 1024;
  constexpr bool kNormRoom = kNormOff + WN * BM * 4 <= kStages * kStage;
  float *norm_x = reinterpret_cast<float *>(lds + kNormOff);
  const bool norm_in = kNormRoom && (EPI == kEpiSwiglu || is_rope(EPI)) && na.ss_in != nullptr;     // uniform
  const bool norm_out = kNormRoom && kWholeRows && EPI == kEpiResidual && na.ss_out != nullptr;                         // uniform
  if (norm_in) {
    if (tid < BM) norm_x[tid] = my_rnorm;
    __syncthreads();
  }
  const int rope_third = is_rope(EPI) ? (tile_n * BN) / (N_out / 3) : 2;   // 0 = q, 1 = k, 2 = v (uniform per workgroup)
  // v third of the QKV projection: a wave keeps two passes (64 keys) in its staging area, so that the
  // key-contiguous copy is written in whole 128-byte lines; columns are XOR-swizzled by the 16-key block
  // of the row, which makes the transposing 2-byte reads free of bank conflicts.
  constexpr int kVPasses = (is_rope(EPI) && WTM % 64 == 0) ? 2 : 1;
  static_assert(WM * WN * kVPasses * 32 * kStride <= kStages * kStage, "v staging area exceeds the LDS ring");
  static_assert(!kNormRoom || WM * WN * kVPasses * 32 * kStride <= kNormOff, "staging area reaches into the norm exchange area");
  const bool v_tile = is_rope(EPI) && rope_third == 2;
  unsigned char *my = lds + wave * ((v_tile ? kVPasses : 1) * 32 * kStride);
  // rotary epilogue: cos / sin of the lane's rows (2 halves of 16) and columns (2 sub-tiles x 4 pairs) of a
  // pass, requested one pass ahead
  const int rope_g = wn & 1;
  float4 csr[is_rope(EPI) ? 2 : 1][2][2][2];
  auto load_cs = [&](int mt) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const int m = m0 + wm * WTM + mt * 32 + h * 16 + fr;
        int pos = EPI == kEpiQkvRopeWin ? ra.row_pos[min(m, M - 1)] : min(m, M - 1) % ra.T;
        if (EPI == kEpiQkvRopeWin && pos < 0) pos = ra.T - 1;
        const float4 *cs4 = reinterpret_cast<const float4 *>(ra.cos_sin + (int64_t)pos * 64 + rope_g * 32 + nt * 16 + 4 * fq);
        csr[is_rope(EPI) ? mt & 1 : 0][h][nt][0] = cs4[0];
        csr[is_rope(EPI) ? mt & 1 : 0][h][nt][1] = cs4[1];
      }
  };
  if (is_rope(EPI) && rope_third < 2) load_cs(0);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (is_rope(EPI) && rope_third < 2 && mt + 1 < MT) load_cs(mt + 1);
    // lane: row h*16 + lane%16 of the pass (h = 16-row half), 4 consecutive columns per n sub-tile
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (2 * mt + h >= MT16) continue;                                 // a last pass of 16 rows
      const int vp = v_tile ? mt % kVPasses : 0;                        // pass inside the v staging group
      unsigned char *wrow = my + (vp * 32 + h * 16 + fr) * kStride;
      const int xs = v_tile ? (2 * vp + h) << 3 : 0;                    // column swizzle of this 16-row block
      const int m16 = 2 * mt + h;
      if (norm_in) {                                                     // row m16 * 16 + fr of the wave tile
        const float rs = norm_x[wm * WTM + m16 * 16 + fr];
#pragma unroll
        for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[nt][m16][e] *= rs;
      }
      if (is_rope(EPI) && rope_third < 2) {
        // a = column i of the head (sub-tile nt), b = column i + 64 (sub-tile nt + 2), both rounded to bf16 first
        // (the values a separate rotary pass would read): i <- a cos - b sin, i + 64 <- b cos + a sin
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          constexpr int kHalf = NT16 / 2;                     // 2 here; keeps the index valid in the other instances
          const int nb = nt % kHalf + kHalf;
          const uint32_t aw[2] = {pack_bf16x2(acc[nt % kHalf][m16][0], acc[nt % kHalf][m16][1]), pack_bf16x2(acc[nt % kHalf][m16][2], acc[nt % kHalf][m16][3])};
          const uint32_t bw[2] = {pack_bf16x2(acc[nb][m16][0], acc[nb][m16][1]), pack_bf16x2(acc[nb][m16][2], acc[nb][m16][3])};
          uint32_t lo[2], up[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float4 c4 = csr[is_rope(EPI) ? mt & 1 : 0][h][nt][e];
            const float a0 = __uint_as_float(aw[e] << 16), a1 = __uint_as_float(aw[e] & 0xffff0000u);
            const float b0 = __uint_as_float(bw[e] << 16), b1 = __uint_as_float(bw[e] & 0xffff0000u);
            const float2 r0 = rotate_pair(a0, b0, c4.x, c4.y), r1 = rotate_pair(a1, b1, c4.z, c4.w);
            lo[e] = pack_bf16x2(r0.x, r1.x);
            up[e] = pack_bf16x2(r0.y, r1.y);
          }
          *reinterpret_cast<uint2 *>(wrow + (nt * 16 + 4 * fq) * 2) = make_uint2(lo[0], lo[1]);
          *reinterpret_cast<uint2 *>(wrow + (32 + nt * 16 + 4 * fq) * 2) = make_uint2(up[0], up[1]);
        }
      } else if (EPI == kEpiSwiglu) {
#pragma unroll
        for (int c = 0; c < NT16 / 2; ++c) {                  // gate sub-tile c, up sub-tile NT16/2 + c
          float v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = silu_f(acc[c][m16][j]) * acc[NT16 / 2 + c][m16][j];
          *reinterpret_cast<uint2 *>(wrow + (c * 16 + 4 * fq) * 2) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
      } else {
#pragma unroll
        for (int nt = 0; nt < NT16; ++nt) {
          const int col = (nt * 16 + 4 * fq) ^ xs;
          if (kStageF32)
            *reinterpret_cast<float4 *>(wrow + col * 4) = make_float4(acc[nt][m16][0], acc[nt][m16][1], acc[nt][m16][2], acc[nt][m16][3]);
          else
            *reinterpret_cast<uint2 *>(wrow + col * 2) = make_uint2(pack_bf16x2(acc[nt][m16][0], acc[nt][m16][1]),
                                                                   pack_bf16x2(acc[nt][m16][2], acc[nt][m16][3]));
        }
      }
    }
    if (is_rope(EPI)) {
      static_assert(!is_rope(EPI) || (WTN == 64 && WN % 2 == 0), "a head is two wave tiles wide");
      const int d_model = N_out / 3;
      const int m_base = m0 + wm * WTM + mt * 32;
      if (rope_third < 2) {
        // staged row: 32 columns from 32g of the head, then the 32 from 64 + 32g
        const int col = tile_n * BN + (wn >> 1) * 128 + rope_g * 32 + (rd_col0 < 32 ? rd_col0 : rd_col0 + 32);
#pragma unroll
        for (int j = 0; j < 32 / kRowsPerInstr; ++j) {
          const int r = j * kRowsPerInstr + rd_row;
          const int m = m_base + r;
          if (m < M) *reinterpret_cast<uint4 *>(C + (int64_t)m * N_out + col) =
                         *reinterpret_cast<const uint4 *>(my + r * kStride + rd_col0 * 2);
        }
      } else {
        const int vp = mt % kVPasses;
        if (ra.store_v)
#pragma unroll
        for (int j = 0; j < 32 / kRowsPerInstr; ++j) {               // v as it is ...
          const int r = j * kRowsPerInstr + rd_row;
          const int rl = vp * 32 + r;                                // row inside the staging group
          const int m = m_base + r;
          if (m < M) *reinterpret_cast<uint4 *>(C + (int64_t)m * N_out + out_col0 + rd_col0) =
                         *reinterpret_cast<const uint4 *>(my + rl * kStride + ((rd_col0 ^ ((rl >> 4) << 3)) * 2));
        }
        // ... and key-contiguous, once the group's passes are staged: a lane gathers the 8 keys of one 16-byte
        // chunk of one d column (each 16 keys are stored as {0-3, 8-11 | 4-7, 12-15}); the lanes of a store
        // cover all chunks of 64 / chunks neighbouring columns
        const int key0 = m_base - vp * 32;
        if ((vp == kVPasses - 1 || mt == MT - 1) && key0 < M) {
          const int vcol0 = out_col0 - 2 * d_model;                  // column inside the v third; 64 columns of one head
          bf16_t *vt_head = ra.vt + (int64_t)(vcol0 & 127) * ra.Tv;
          const int per_seq = EPI == kEpiQkvRopeWin ? ra.R : ra.T;   // rows a canvas
          if (EPI == kEpiQkvRopeWin || ra.T % 16 == 0) {
            const int chunks = 4 * (vp + 1);                         // 16-byte chunks per column: 4 or 8
            const int g = lane % chunks, blk = g >> 1;
            int seq = key0 / per_seq, t0 = key0 % per_seq + 16 * blk;
            if (per_seq % 64 != 0) { seq = (key0 + 16 * blk) / per_seq; t0 = (key0 + 16 * blk) % per_seq; }   // a group of 64 keys may straddle canvases
            const unsigned char *src = my + (16 * blk + 4 * (g & 1)) * kStride;
            bf16_t *dst = vt_head + ((int64_t)seq * ra.H + (vcol0 >> 7)) * 128 * ra.Tv + t0 + (g & 1) * 8;
            if (key0 + 16 * blk < M)
#pragma unroll
            for (int it = 0; it < chunks; ++it) {
              const int c = it * (64 / chunks) + lane / chunks;
              const unsigned char *sc = src + ((c ^ (blk << 3)) * 2);
              uint32_t w[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {                          // key pairs (0,1) (2,3) (8,9) (10,11) of the chunk's half
                const int kr = (e & 1) * 2 + (e >> 1) * 8;
                const uint32_t lo = *reinterpret_cast<const uint16_t *>(sc + kr * kStride);
                const uint32_t hi = *reinterpret_cast<const uint16_t *>(sc + (kr + 1) * kStride);
                w[e] = lo | (hi << 16);
              }
              *reinterpret_cast<uint4 *>(dst + (int64_t)c * ra.Tv) = make_uint4(w[0], w[1], w[2], w[3]);
            }
          } else {
            const int keys = 32 * (vp + 1);                          // lane = key; 4 columns per LDS read
            const int key = lane % keys, m = key0 + key;
            if (m < M) {
              const int seq = m / per_seq, t = m % per_seq;
              const unsigned char *src = my + key * kStride;
              bf16_t *dst = vt_head + ((int64_t)seq * ra.H + (vcol0 >> 7)) * 128 * ra.Tv + ((t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1));
#pragma unroll 4
              for (int c = 4 * (lane / keys); c < 64; c += 4 * (64 / keys)) {
                const uint2 x = *reinterpret_cast<const uint2 *>(src + ((c ^ ((key >> 4) << 3)) * 2));
                const uint32_t w[4] = {x.x & 0xffffu, x.x >> 16, x.y & 0xffffu, x.y >> 16};
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(int64_t)(c + e) * ra.Tv] = __builtin_bit_cast(bf16_t, (uint16_t)w[e]);
              }
            }
          }
        }
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < kRowIters; ++j) {
      const int r = st_row(j), rd_col = st_col(j);
      if (WTM % 32 != 0 && mt * 32 + (kWholeRows ? j * kRowsPerInstr : r) >= WTM) continue;      // beyond a last pass of 16 rows
      const int m = m0 + wm * WTM + mt * 32 + r;
      const int64_t o = (int64_t)m * N_out + out_col0 + rd_col;
      if (EPI == kEpiPartial) {
        if (m < M) {
          float4 *dst = reinterpret_cast<float4 *>(sk.partial + (int64_t)blockIdx.y * M * N_out + o);
          dst[0] = *reinterpret_cast<const float4 *>(my + r * kStride + rd_col * 4);
          dst[1] = *reinterpret_cast<const float4 *>(my + r * kStride + rd_col * 4 + 16);
        }
        continue;
      }
      uint4 out;
      if (EPI == kEpiResidual) {
        const float4 x0 = *reinterpret_cast<const float4 *>(my + r * kStride + rd_col * 4);
        const float4 x1 = *reinterpret_cast<const float4 *>(my + r * kStride + rd_col * 4 + 16);
        const uint4 r4 = rs[EPI == kEpiResidual ? mt : 0][j];
        out.x = pack_bf16x2(x0.x + __uint_as_float(r4.x << 16), x0.y + __uint_as_float(r4.x & 0xffff0000u));
        out.y = pack_bf16x2(x0.z + __uint_as_float(r4.y << 16), x0.w + __uint_as_float(r4.y & 0xffff0000u));
        out.z = pack_bf16x2(x1.x + __uint_as_float(r4.z << 16), x1.y + __uint_as_float(r4.z & 0xffff0000u));
        out.w = pack_bf16x2(x1.z + __uint_as_float(r4.w << 16), x1.w + __uint_as_float(r4.w & 0xffff0000u));
      } else {
        out = *reinterpret_cast<const uint4 *>(my + r * kStride + rd_col * 2);
      }
      if (m < M) *reinterpret_cast<uint4 *>(C + o) = out;
      if (norm_out) {                                                    // sum of squares of the row's rounded values
        const uint32_t ow[4] = {out.x, out.y, out.z, out.w};
        float q = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = __uint_as_float(ow[e] << 16), b = __uint_as_float(ow[e] & 0xffff0000u);
          q += a * a + b * b;
        }
#pragma unroll
        for (int off = 1; off < LPR; off <<= 1) q += __shfl_xor(q, off, 64);   // the LPR lanes that share the row
        if (rd_col == 0) norm_x[wn * BM + wm * WTM + mt * 32 + r] = q;
      }
    }
  }
  if (norm_out) {
    // The sums of 64 columns, from left to right: a slot of 256, or slots of 64 where the tile is narrower (its reader adds four
    // of them first), so that a row's sum is the same bits whatever tile shape the launch took.
    constexpr int kPerSlot = BN == 256 ? 256 : 64, kSlots = BN / kPerSlot, kWaves64 = WTN < 64 ? 64 / WTN : 1;
    static_assert(EPI != kEpiResidual || WTN == 64 || WTN == 32, "64 columns are whole waves");
    __syncthreads();
    for (int row = tid; row < BM; row += kThreads) {
      if (m0 + row >= M) continue;
#pragma unroll
      for (int sl = 0; sl < kSlots; ++sl) {
        float t = 0.f;
#pragma unroll
        for (int c = 0; c < kPerSlot / 64; ++c) {
          const float *x = norm_x + (sl * (kPerSlot / 64) + c) * kWaves64 * BM + row;
          t += kWaves64 == 2 ? x[0] + x[BM] : x[0];
        }
        na.ss_out[((int64_t)tile_n * kSlots + sl) * na.ld + m0 + row] = t;
      }
    }
  }
}

template <int EPI, int BM, int BN, int BK, int ST, int WM, int WN, bool kPairs = true>
pvf_status run(pvf_ctx *ctx, hipStream_t s, const void *A, const void *W, void *C, const void *Res,
               int M, int N_out, int K, const RopeArgs &ra, const SplitK &split = SplitK{nullptr, 0}, int splits = 1,
               const NormArgs &na = NormArgs{}) {
  constexpr int kLdsBytes = ST * (BM + BN) * BK * 2;
  static_assert(kLdsBytes <= 160 * 1024, "LDS ring exceeds the 160 KB of a CU");
  const int tiles_m = (M + BM - 1) / BM;
  const int tiles_n = (EPI == kEpiSwiglu) ? N_out / (BN / 2) : N_out / BN;
  const int total = tiles_m * tiles_n;
  // bands of at most kBand tile rows, all of (nearly) the same height: the 32 workgroups that run
  // together on an XCD then cover a patch of kBand x 32/kBand tiles in every band, whose operand rows
  // that XCD's L2 fetches once.  The patch that fetches least has rows : columns = BN : BM.
  constexpr int kBand = BM > BN ? 4 : 8;
  const int n_bands = (tiles_m + kBand - 1) / kBand;
  const int group_m = (tiles_m + n_bands - 1) / n_bands;
  // Workgroups that touch weights ahead on the CUs of the last round that have no tile (touch_weights).  They read as fast as a tile's
  // own loads go (47 GB/s a CU), so they take all stages where that ends before the tiles do (in_time, in eighths), every second one
  // where half of it does, and none otherwise: every third or fourth is slower than none.  K = 4096 unless noted: QKV of 128
  // rows 29.8 -> 28.6 us, 384 47.2 -> 44.2, 512 55.5 -> 48.2; gate/up of 2 x 12288 columns, 128 rows 46.1 -> 42.0, 192 53.5 -> 49.8, 2 x
  // 9216, K = 3072, 256 rows 49.7 -> 40.0; O of 768 rows 37.9 -> 32.6, down (K = 12288) 111 -> 86, of 1311 rows 132 -> 124.  Not up to 64
  // rows, which HBM itself bounds (33 rows of 9216 columns, K = 3072, 15.4 -> 17.4); not with weights below 16 MB, which most tiles find in L2
  // (1311 rows of 1024 columns, K = 2048, 14.7 -> 15.6); not behind tiles of 256 x 256, which the MFMAs bound (1024 rows 80-85 either way).
  // Shapes of which two tiles fit a CU (64 x 64 and 64 x 128 rings of up to 80 KB) are counted like the others: the tiles past 32 of an
  // XCD start at once, but on a CU that has one already, and gain by it.  K = 4096, without and with: 192 rows of 12416 columns 53.5 -> 49.7
  // us, of 2 x 6208 54.2 -> 49.8, 128 rows of 9216 37.4 -> 33.4, 256 rows of 17280 (68 tiles) 83.4 -> 74.1; the other side, 192 rows of 11008
  // (33 tiles) 40.0 -> 41.1 and 256 rows of 8832 46.0 -> 46.8.
  const int chunk = (total + 7) / 8, in_last = chunk % 32, idle = 32 - in_last;     // tiles and idle CUs of an XCD in the last round
  const int w_rows = EPI == kEpiSwiglu ? 2 * N_out : N_out;
  SplitK sk = split;
  if (touches(EPI, BM, BN) && M > 64 && in_last > 0 && idle >= 4 && K >= 1024 && (int64_t)w_rows * K >= 8 << 20) {
    const int rows = std::min(tiles_m, group_m), n_cols = 1 + (in_last + rows - 2) / rows;       // at most
    sk.ahead = std::min(idle, n_cols);
    const int in_time = 32 * (BM + BN) / (5 * BN * ((n_cols + sk.ahead - 1) / sk.ahead));
    sk.ahead8 = in_time >= 8 ? 8 : 4;
    if (in_time < 4) sk.ahead = 0;
  }
  const int grid = 8 * (chunk + sk.ahead);
  auto launch = [&](auto hint, auto turn) -> pvf_status {
    const auto kernel = gemm_bf16_mfma_kernel<EPI, BM, BN, BK, ST, WM, WN, kPairs, decltype(hint)::value, decltype(turn)::value>;
    // once per kernel instance; a function-local static is initialised exactly once even with concurrent callers
    static const hipError_t configured =
        hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    PVF_HIP_CHECK(ctx, configured);
    kernel<<<dim3(grid, splits), 64 * WM * WN, kLdsBytes, s>>>(
        (const bf16_t *)A, (const bf16_t *)W, (bf16_t *)C, (const bf16_t *)Res, M, N_out, K, tiles_m, tiles_n, group_m, ra, sk, na);
    PVF_LAUNCH_CHECK(ctx, "gemm_mfma");
    return PVF_OK;
  };
  // Weights that at most two rows of tiles read are loaded with the non-temporal hint by the shapes that gain, so that they do not
  // push the activations and the partial sums out of L2 (cached rounds of 64 and 320 rows 4.4 and 2.5 % faster).  With more rows of
  // tiles they may be gone before the last one reads them: 160 x 256 tiles at 1311 rows of 6144 columns, K = 2048, 40.1 us with the
  // hint and 34.4 without, K = 8192 132 and 121; 4100 rows of 12288 columns, K = 4096, 352 and 335.
  // shapes for at most two rows of tiles (160 x 192: a forced shape aside)
  constexpr bool kFewRows = EPI == kEpiPartial ? BM == 64 : BN == 64 || ST == 6 || (EPI == kEpiSwiglu && BM == 160);
  constexpr bool kTwoRows = (EPI == kEpiPartial && BN == 192) || (EPI == kEpiStore && BM == 160);
  // shapes that the launches taking the whole of K behind few rows are made of
  constexpr bool kTurns = ((EPI == kEpiStore || EPI == kEpiQkvWindow) && BN == 64) || (EPI == kEpiSwiglu && BN == 128 && (ST == 6 || BM == 128)) ||
                          (EPI == kEpiSwiglu && kPairs && (BM == 192 || BM == 160 || (BM == 256 && BN == 128))) || (EPI == kEpiStore && BM == 192 && BN == 128);
  if constexpr (kTurns) if (sk.turn) return launch(std::bool_constant<kFewRows>{}, std::true_type{});
  if constexpr (kFewRows) return launch(std::true_type{}, std::false_type{});
  else {
    if constexpr (kTwoRows) if (tiles_m <= 2) return launch(std::true_type{}, std::false_type{});
    return launch(std::false_type{}, std::false_type{});
  }
}

struct TileCfg { int bm, bn, bk, stages; double eff; bool plain_only, pairs_only = false; };   // pairs_only: SwiGLU with K % 128 == 0 (the quadrant schedule)
constexpr int kNumCfg = 14;
// Every shape for many rows runs 8 waves, two per SIMD (the two small ones 4 waves, two workgroups per CU):
// with one wave per SIMD the 256 x 256 tile (wave tiles of 128 x 128, a third fewer LDS reads) measured 2-4 %
// slower, smaller wave tiles far slower.
// plain_only: wave tiles 32 columns wide, which the rotary epilogue cannot pair up, or 80 rows high (a last epilogue pass of 16
// rows, which only the plain epilogues handle).  SwiGLU takes 192 x 128 among them (16 gate and 16 up columns a wave), by
// few_rows_shape alone.
constexpr TileCfg kCfg[kNumCfg] = {
    {256, 256, 64, 2, 1.00, false},   // the wide layers
    {128, 256, 64, 3, 0.89, false}, {256, 128, 64, 3, 0.891, false},
    {128, 128, 64, 5, 0.70, false},   // launches of a single round of tiles: the smallest area finishes first
    {192, 256, 64, 2, 0.94, false},   // fills the chip when M / 256 leaves many CUs idle
    {320, 128, 64, 2, 0.78, true},    // 2560 rows = 8 tile rows: with N = 4096 exactly one tile per CU (wave tiles 80 x 64)
    {64, 64, 64, 5, 0.0, true},       // few rows (window forward of the K/V-cached rounds): the GEMM streams the weights;
    {64, 128, 64, 3, 0.0, false},     // these two and the last two are chosen by pick_config for M <= 384
    {192, 128, 64, 3, 0.86, true},    // 1536 rows = 8 tile rows: with N = 4096 one tile per CU; SwiGLU of 129-192 rows (pick_config)
    {160, 256, 64, 3, 0.85, true},   // 2560 rows = 16 tile rows: one tile per CU like 320 x 128, with room for a third stage
    {256, 192, 64, 2, 0.965, false, true},   // gate/up of 24576 weight rows = 128 tile columns: 512 rows are one tile per CU
    {64, 128, 64, 6, 0.0, false}, {128, 64, 64, 6, 0.0, true},   // the whole of K behind one workgroup a CU: rings of 144 KB
    {160, 192, 64, 3, 0.0, true}};                               // SwiGLU of 257-320 rows (swiglu_160x192_pays)

template <int EPI>
pvf_status run_cfg(pvf_ctx *ctx, hipStream_t s, int cfg, const void *A, const void *W, void *C,
                   const void *Res, int M, int N, int K, const RopeArgs &ra = RopeArgs{}, const NormArgs &na = NormArgs{}, bool turn = false) {
  const SplitK whole{nullptr, 0, turn && (M <= 128 ? K >= 1024 : M <= 384 && K >= 2048)};
  constexpr bool kPlain = EPI != kEpiSwiglu && !is_rope(EPI);
  if (K % 128 != 0 && cfg == 0) return run<EPI, 256, 256, 64, 2, 2, 4, false>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na);
  if (K % 128 != 0 && cfg == 4) return run<EPI, 192, 256, 64, 2, 2, 4, false>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na);
  switch (cfg) {
    case 0: return run<EPI, 256, 256, 64, 2, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na);
    case 1: return run<EPI, 128, 256, 64, 3, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na);
    case 2: return run<EPI, 256, 128, 64, 3, 4, 2>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na);
    case 4: return run<EPI, 192, 256, 64, 2, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na);
    case 5: if constexpr (kPlain) return run<EPI, 320, 128, 64, 2, 4, 2>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na); break;
    case 6: if constexpr (kPlain) return run<EPI, 64, 64, 64, 5, 2, 2>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na); break;
    case 7: return run<EPI, 64, 128, 64, 3, 2, 2>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na);
    case 8: if constexpr (!is_rope(EPI)) return run<EPI, 192, 128, 64, 3, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na); break;
    case 9: if constexpr (kPlain) return run<EPI, 160, 256, 64, 3, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na); break;
    case 10: if constexpr (EPI == kEpiSwiglu) return run<EPI, 256, 192, 64, 2, 4, 2>(ctx, s, A, W, C, Res, M, N, K, ra, SplitK{nullptr, 0}, 1, na); break;
    case 11: if constexpr (EPI == kEpiSwiglu) return run<EPI, 64, 128, 64, 6, 2, 2>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na); break;
    case 13: if constexpr (EPI == kEpiSwiglu) return run<EPI, 160, 192, 64, 3, 2, 4>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na); break;
    case 12: if constexpr (EPI == kEpiStore) return run<EPI, 128, 64, 64, 6, 4, 2>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na); break;
    default: break;
  }
  return run<EPI, 128, 128, 64, 5, 4, 2>(ctx, s, A, W, C, Res, M, N, K, ra, whole, 1, na);
}

// Gate/up of 257-320 rows on two rows of 160 x 192 tiles over the whole of K.  By times of both ways at 264 and 320 rows, N = 1536-24576
// and K = 512-8192 (320 rows here): where the tiles make most of a round, or the loop is short.  2 x 12288 columns, K = 4096,
// 68.3 us divided and 58.3 whole; 9216, K = 8192, 113 and 106, K = 1024 30.8 and 19.2; 24576, K = 4096, 196 (64 x 128 tiles) and 122.  The
// other side: 7680, K = 8192, 88 and 102; 6144, K = 4096, 44.6 and 54.0; 4608, K = 2048, 29.2 and 30.0; 13824 (a second round for a
// few), K = 1024, 36.6 and 36.9.
bool swiglu_160x192_pays(int N, int K) {
  if (N % 96 != 0) return false;
  const int tiles = N / 48;
  if (tiles > 256) return N > 16384 || K <= 512 || (tiles >= 320 && K <= 1024);      // wider than 2 x 16384: K is not divided
  return tiles >= 192 || K <= (tiles >= 160 ? 4096 : tiles >= 128 ? 2048 : tiles >= 64 ? 1024 : 0);
}

// Undivided shapes for few rows; -1: by the estimate.  Up to 128 rows rings of 5-6 stages (64-120 KB of weights on the way per CU) where
// the tiles, one a CU, make one round or the loop is long: 96 rows of 20480 columns, K = 1024, 17.4 us on 128 x 64 and 14.8 on 64 x 64,
// two a CU; 32 rows of gate/up 2 x 20480, K = 512, 14.4 on six stages and 11.7 on three.  From there tiles as tall as the launch or
// half of it.
int few_rows_shape(GemmEpilogue epi, int M, int N, int K) {
  if (M > 384) return -1;
  if (epi == kEpiSwiglu) {
    if (M <= 64) return N >= 9216 && (N <= 16384 || K >= 2048) ? 11 : 7;
    if (M <= 128) return N >= 8192 && K >= (N <= 16384 ? 1024 : 2048) ? 3 : 7;
    if (M > 256 && M <= 320 && swiglu_160x192_pays(N, K)) return 13;
    if (N < 8192 || N > 16384 || N % 128 != 0 || (M > 256 && M <= 320)) return 7;
    return M <= 192 ? 8 : M <= 256 ? 2 : 4;
  }
  if (epi == kEpiStore && M > 64 && M <= 128 && N > 8192 && N % 64 == 0 && (N <= 16384 || N > 24576 || K >= 4096)) return 12;
  if (epi != kEpiQkvRope && M <= 128 && N % 64 == 0) return 6;
  return epi == kEpiStore && M > 320 && N >= 8192 && N <= 16384 && N % 128 == 0 ? 8 : N % 128 == 0 ? 7 : -1;
}
// Whether a launch of few rows that could divide K takes the whole of it: it then writes bf16 once instead of float32 partial sums
// that another launch adds up, but has no more workgroups than tiles (wgs), and each of them a longer loop.  By times of both ways
// at K = 512-12288 and N = 4096-32768: whole where the tiles make most of a round, or the loop is short.  At K = 4096:
// 64 rows, QKV of 12288 columns 33.5 -> 22.9 us, gate/up of 2 x 12288 46.8 -> 35.5; 160 rows, gate/up 63 -> 56, 384 rows 103 -> 78, QKV
// 55 -> 49.  The other side of the limits: 64 rows of 6144 columns, K = 8192, 29 us divided and 37 whole; gate/up of 2 x 8192, K = 3072,
// 160 rows 34.5 and 40.8; 384 rows of 8192 columns, K = 8192, 62 and 86; gate/up of 2 x 9216, K = 8192, 384 rows 130 and 137.
bool takes_whole_k(GemmEpilogue epi, int M, int N, int K) {
  const int wgs = N / 64;                          // of every shape below but the 64 x 64 tiles of 65-128 rows
  if (epi == kEpiSwiglu) {
    if (M <= 64) return wgs >= 144;
    if (M <= 128) return wgs >= 144 || (wgs >= 128 && K >= 1024 && K <= 2048);
    if (M > 256 && M <= 320) return swiglu_160x192_pays(N, K);
    if (M > 384 || wgs < 128 || wgs > 256 || N % 128 != 0) return false;
    if (wgs < 144 || K <= 1024) return K <= 1024;
    if (M <= 192) return K <= (wgs < 256 ? 8192 : 3072);       // 256: gate and up columns a power of two apart, 6-15 % slower from K = 4096 on
    if (M <= 256) return K <= (wgs < 160 ? 4096 : wgs < 224 ? 8192 : INT_MAX);
    return wgs >= 172 || K <= 2048;
  }
  if (epi != kEpiStore) return false;
  if (M <= 64) return N % 64 == 0 && wgs >= 96 && (wgs >= 144 || K <= 2048);
  if (M <= 128) return N % 64 == 0 && wgs >= 96 && K <= (wgs >= 256 ? 8192 : 4096);
  return M > 320 && M <= 384 && N % 128 == 0 && wgs >= 128 && wgs <= 256 && (wgs >= 192 || K <= 2048);
}

// Tile shape: the one with the least estimated time = rounds of workgroups over the 256 CUs
// x tile area / relative efficiency of the shape (measured on the forward's GEMM shapes: the
// smaller tiles re-read operands more often but quantise better when there are few tiles).  What a last round leaves idle is lost in
// launches of one or two rounds and counts for less behind several, whose workgroups no longer end together: a tenth of it is given
// back per round before it, at most 0.4.  Shares and efficiencies follow the times of every shape on 17 matrices of 2048-24576 columns
// and K = 2048-13824 at 34 numbers of rows from 385 to 4100.  Whole rounds alone: 0.5 % slower on average (gate/up of 2 x 12288, K =
// 4096, 1311 rows, 230 against 219 us, 3.0 rounds of 256 x 192 tiles and 2.6 of 192 x 256; 2304 rows of 24576 columns, K = 8192, 819
// against 687).  0.4 of the idle part given back in every round: 0.2 % on average and up to 11 % (gate/up of 2 x 14336, K = 4096, 640
// rows, 165 against 149; 1792 rows of 12288 columns, K = 4096, 162 against 146).
// PVF_GEMM_TILE=<n> in the environment forces shape n (for tuning runs).
int pick_config(GemmEpilogue epi, int M, int N, int K, double *cost = nullptr) {
  static const int forced = [] { const char *e = getenv("PVF_GEMM_TILE"); return (e && e[0]) ? atoi(e) : -1; }();
  const bool plain = epi != kEpiSwiglu && epi != kEpiQkvRope;
  // Few rows: the launch streams the weight matrix once and is bound by HBM, not by the MFMAs.
  // Many small workgroups with deep LDS rings keep more bytes in flight (measured on the layer
  // shapes: 3.2x faster than the large tiles at M = 64, 2x at M = 320).
  // The output head (N = vocabulary) has enough tiles to fill the chip at any M > 64 and goes by the
  // cost model below.
  if (forced < 0 && M <= 384 && (M <= 64 || N <= 32768)) {
    const int c = few_rows_shape(epi, M, N, K);
    if (c >= 0) return c;
  }
  int best = -1;
  double best_t = 0;
  for (int c = 0; c < kNumCfg; ++c) {
    const int ncols = (epi == kEpiSwiglu) ? kCfg[c].bn / 2 : kCfg[c].bn;
    if (N % ncols != 0 || K % kCfg[c].bk != 0 || (kCfg[c].plain_only && !plain) || (kCfg[c].pairs_only && (epi != kEpiSwiglu || K % 128 != 0))) continue;
    if (forced == c) return c;
    if (kCfg[c].eff <= 0.0) continue;
    const int64_t tiles = (int64_t)((M + kCfg[c].bm - 1) / kCfg[c].bm) * (N / ncols);
    // two rows of tiles at most: what counts is by how many rows of tiles the weights are read (512 rows, QKV of 12288 columns:
    // 128 x 256 60.5 us, 256 x 128 54.6)
    // Above, a residual projection also writes the rows' sums of squares, four times as many from 128 columns as from 256, and the
    // projection behind it reads them: 256 x 128 before 128 x 256 there gains 5-9 % of the down projection and loses more (5 x 320
    // tokens 22.0 -> 22.5 ms).
    const double eff = c == 2 && M <= 512 ? 0.95 : c == 2 && epi == kEpiResidual ? 0.885 : kCfg[c].eff;
    const double full = (double)tiles / 256, rounds = (double)((tiles + 255) / 256);
    const double back = std::min(0.02 + 0.1 * (rounds - 1), 0.4);      // 0.02: of equal rounds the fewer tiles
    const double t = (rounds - back * (rounds - full)) * kCfg[c].bm * kCfg[c].bn / eff;
    if (best < 0 || t < best_t) { best = c; best_t = t; }
  }
  if (cost) *cost = best_t;
  return best;
}

// Adds the partial sums of a split-K launch in split order (deterministic) and finishes like the
// fused epilogues: store, + residual (rounded once), or SwiGLU of the gate | up halves of a partial row.
// One thread = 8 consecutive output columns of one row.  Nw = length of a partial row.
template <int EPI>
__global__ void __launch_bounds__(256)
splitk_finalize_kernel(const float *__restrict__ partial, int splits, int M, int Nw, int N_out,
                       bf16_t *__restrict__ out, const bf16_t *__restrict__ res) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int per_row = N_out / 8;
  if (idx >= (int64_t)M * per_row) return;
  const int m = (int)(idx / per_row), c = (int)(idx % per_row) * 8;
  float v[8], u[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = u[e] = 0.f;
  for (int z = 0; z < splits; ++z) {
    const float *row = partial + ((int64_t)z * M + m) * Nw + c;
    const float4 a0 = *reinterpret_cast<const float4 *>(row), a1 = *reinterpret_cast<const float4 *>(row + 4);
    v[0] += a0.x; v[1] += a0.y; v[2] += a0.z; v[3] += a0.w; v[4] += a1.x; v[5] += a1.y; v[6] += a1.z; v[7] += a1.w;
    if (EPI == kEpiSwiglu) {
      const float4 b0 = *reinterpret_cast<const float4 *>(row + N_out), b1 = *reinterpret_cast<const float4 *>(row + N_out + 4);
      u[0] += b0.x; u[1] += b0.y; u[2] += b0.z; u[3] += b0.w; u[4] += b1.x; u[5] += b1.y; u[6] += b1.z; u[7] += b1.w;
    }
  }
  if (EPI == kEpiSwiglu) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = silu_f(v[e]) * u[e];
  }
  const int64_t o = (int64_t)m * N_out + c;
  if (EPI == kEpiResidual) {
    const uint4 rs = *reinterpret_cast<const uint4 *>(res + o);
    const uint32_t rw[4] = {rs.x, rs.y, rs.z, rs.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] += __uint_as_float(rw[e] << 16);
      v[2 * e + 1] += __uint_as_float(rw[e] & 0xffff0000u);
    }
  }
  *reinterpret_cast<uint4 *>(out + o) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                   pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

constexpr int kSplitMaxRows = 640;   // launches with more rows have enough tiles without splitting K

// Tile shape and number of splits of a split-K launch; splits = 0: not possible.
//  up to 64 rows  64 x 64 with five stages, up to one workgroup per CU, two where K is divided in two: fewer partial sums than 64 x 128 with two workgroups a CU
//                 (O projection with its reduction 16.4 -> 13.0 us, down 26.5 -> 24.5)
//  above          the shapes below by estimated time: rounds of workgroups over the chip x (k stages per workgroup + ~8
//                 stages' worth of prologue and epilogue) x the tile's area over its relative efficiency, plus what the
//                 partial sums cost, 4 bytes written and read per split and element.  Which shapes stand against each other in a
//                 range of rows, and their efficiencies, follow the times of the O (K = 4096) and down (12288) projections of 4096
//                 columns.  96 rows: O 64 x 64 in 2 15.1 us, 128 x 128 in 8 17.6; down 33 (64 x 64), 28.6.  192 rows: O 128 x 128
//                 in 4 19.9, 192 x 128 in 8 23.6; down 36.9, 34.3.  256 rows: O 128 x 128 in 4 22.2, 256 x 128 in 8 26.0; down 42.1,
//                 39.6.  512 rows: O 128 x 128 in 2 29.3; down 67.6, 256 x 128 in 4 57.9.  640 rows: O 160 x 128 in 2 32.8, undivided
//                 35.4; down 160 x 256 in 4 67.8, undivided 108.  193-256 rows of 9216 columns, K = 4096: 160 x 192 in 2 36 us, 256 x
//                 128 in 2 38 (as fast as one another at 4096 columns, which 192 does not divide).
enum SplitTile { kS64x64, kS192x128, kS320x128, kS160x256, kS160x192, kS160x128, kS128x128, kS128x256, kS256x128 };
struct SplitShape { SplitTile tile; int bm, bn; double eff; };
void splitk_plan(int M, int Nw, int K, size_t ws_floats, SplitTile *tile, int *splits) {
  constexpr SplitShape k64[] = {{kS64x64, 64, 64, 1}}, k128[] = {{kS64x64, 64, 64, 0.3}, {kS128x128, 128, 128, 0.66}};
  constexpr SplitShape k192[] = {{kS128x128, 128, 128, 0.66}, {kS192x128, 192, 128, 0.72}};
  constexpr SplitShape k256[] = {{kS128x128, 128, 128, 0.66}, {kS256x128, 256, 128, 1.0}, {kS160x192, 160, 192, 0.97}};
  constexpr SplitShape k384[] = {{kS160x256, 160, 256, 0.85}, {kS160x192, 160, 192, 0.80}, {kS160x128, 160, 128, 0.65},
                                  {kS192x128, 192, 128, 0.72}, {kS320x128, 320, 128, 0.70}};
  constexpr SplitShape k640[] = {{kS128x128, 128, 128, 0.70}, {kS128x256, 128, 256, 0.89}, {kS256x128, 256, 128, 0.93},
                                 {kS160x256, 160, 256, 0.85}, {kS160x128, 160, 128, 0.65}};
  const SplitShape *shapes = M <= 64 ? k64 : M <= 128 ? k128 : M <= 192 ? k192 : M <= 256 ? k256 : M <= 384 ? k384 : k640;
  const int n_shapes = M <= 64 ? 1 : M <= 192 ? 2 : M <= 256 ? 3 : 5, nk = K / 64;
  *tile = shapes[0].tile;
  *splits = 0;
  // 385-640 rows split only where tiles of 128 x 128 would leave half the chip idle or, behind a loop of 64 stages or more, make a
  // second round for a few (the O and down projections: 128-160 tiles).  576 rows of 4096 columns: K = 2048 19.6 us whole and 24-26
  // divided, K = 12288 102 and 67.
  if (M > 384 && (M + 127) / 128 * (Nw / 128) > (K >= 4096 ? 160 : 128)) return;
  double best = 0;
  for (const SplitShape *c = shapes; c < shapes + n_shapes; ++c) {
    if (Nw % c->bn != 0) continue;
    const int64_t tiles = (int64_t)((M + c->bm - 1) / c->bm) * (Nw / c->bn);
    for (int sp = 1; sp <= 8; sp <<= 1) {
      if (nk % sp != 0 || nk / sp < 8 || (size_t)sp * M * Nw > ws_floats) continue;
      // a stage of 160 x 256 takes about 1 us; 5 TB/s for the partial sums
      const double us = M <= 64 ? (tiles * sp <= (sp == 2 ? 512 : 256) ? -sp : 1)
                                : (double)((tiles * sp + 255) / 256) * (nk / sp + 8) * (c->bm * c->bn) / c->eff * 2.1e-5 + sp * (double)M * Nw * 1.6e-6;
      if (*splits == 0 || us < best) { *tile = c->tile; *splits = sp; best = us; }
    }
  }
}

}  // namespace

bool gemm_mfma_supported(int dtype, GemmEpilogue epi, int M, int N, int K);
bool gemm_mfma_norm_capable(int cfg);

// Few rows (window forward of the K/V-cached rounds, full forward of one short canvas): tiles of which one or two
// rows cover the launch, so that every weight row goes from L2 to few CUs, and K split over 2-8 workgroups per tile
// to fill the chip and to shorten the serial k loop; a second small kernel adds the partial sums.  ws: float32 scratch.
bool gemm_mfma_splitk_supported(int dtype, GemmEpilogue epi, int M, int N, int K, size_t ws_floats) {
  if (epi == kEpiQkvRope || epi == kEpiPartial || !gemm_mfma_supported(dtype, epi, M, N, K)) return false;
  const int Nw = epi == kEpiSwiglu ? 2 * N : N;
  if (M > kSplitMaxRows || Nw % 128 != 0 || N % 8 != 0 || Nw > 32768 || takes_whole_k(epi, M, N, K)) return false;
  SplitTile tile;
  int splits;
  splitk_plan(M, Nw, K, ws_floats, &tile, &splits);
  // one split where a launch of its own takes the 64 x 128 tiles (SwiGLU, whose fused epilogue the tall tiles do not have, and
  // wide plain stores)
  return splits >= 2 || (splits == 1 && epi != kEpiResidual && M > 128 && M <= 384);
}

// The split-K launch alone: float32 partial tiles ws[split][M][Nw] (Nw = weight rows: 2 N for SwiGLU); *splits_out
// = number of splits written.
pvf_status launch_gemm_mfma_splitk_partial(pvf_ctx *ctx, hipStream_t s, const void *A, const void *W, int M, int Nw, int K,
                                           float *ws, size_t ws_floats, int *splits_out) {
  const uintptr_t al = (uintptr_t)A | (uintptr_t)W | (uintptr_t)ws;
  PVF_REQUIRE(ctx, (al & 15u) == 0, PVF_EINVAL, "gemm_mfma: operands must be 16-byte aligned");
  SplitTile tile;
  int splits;
  splitk_plan(M, Nw, K, ws_floats, &tile, &splits);
  PVF_REQUIRE(ctx, splits >= 1 && ws != nullptr, PVF_ESHAPE, "gemm_mfma: no split-K plan for M=%d N=%d K=%d", M, Nw, K);
  const SplitK sk{ws, K / 64 / splits};
  *splits_out = splits;
  switch (tile) {
    case kS64x64: return run<kEpiPartial, 64, 64, 64, 5, 2, 2>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS192x128: return run<kEpiPartial, 192, 128, 64, 3, 2, 4>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS320x128: return run<kEpiPartial, 320, 128, 64, 2, 4, 2>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS160x256: return run<kEpiPartial, 160, 256, 64, 3, 2, 4>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS160x192: return run<kEpiPartial, 160, 192, 64, 3, 2, 4>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS160x128: return run<kEpiPartial, 160, 128, 64, 4, 2, 4>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS256x128: return run<kEpiPartial, 256, 128, 64, 3, 4, 2>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS128x128: return run<kEpiPartial, 128, 128, 64, 5, 4, 2>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
    case kS128x256: return run<kEpiPartial, 128, 256, 64, 3, 2, 4>(ctx, s, A, W, nullptr, nullptr, M, Nw, K, RopeArgs{}, sk, splits);
  }
  return PVF_EINVAL;
}

pvf_status launch_splitk_finalize(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const float *partial, int splits,
                                  int M, int N, void *C, const void *residual) {
  const int Nw = epi == kEpiSwiglu ? 2 * N : N;
  const int blocks = (int)(((int64_t)M * (N / 8) + 255) / 256);
  if (blocks == 0) return PVF_OK;
  if (epi == kEpiSwiglu) splitk_finalize_kernel<kEpiSwiglu><<<blocks, 256, 0, s>>>(partial, splits, M, Nw, N, (bf16_t *)C, nullptr);
  else if (epi == kEpiResidual) splitk_finalize_kernel<kEpiResidual><<<blocks, 256, 0, s>>>(partial, splits, M, Nw, N, (bf16_t *)C, (const bf16_t *)residual);
  else splitk_finalize_kernel<kEpiStore><<<blocks, 256, 0, s>>>(partial, splits, M, Nw, N, (bf16_t *)C, nullptr);
  PVF_LAUNCH_CHECK(ctx, "splitk_finalize");
  return PVF_OK;
}

pvf_status launch_gemm_mfma_splitk(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const void *A, const void *W,
                                   void *C, const void *residual, int M, int N, int K, float *ws, size_t ws_floats) {
  const uintptr_t al = (uintptr_t)C | (uintptr_t)residual;
  PVF_REQUIRE(ctx, (al & 15u) == 0, PVF_EINVAL, "gemm_mfma: operands must be 16-byte aligned");
  int splits = 0;
  pvf_status st = launch_gemm_mfma_splitk_partial(ctx, s, A, W, M, epi == kEpiSwiglu ? 2 * N : N, K, ws, ws_floats, &splits);
  if (st != PVF_OK) return st;
  return launch_splitk_finalize(ctx, s, epi, ws, splits, M, N, C, residual);
}


// QKV projection with the rotary embedding and the key-contiguous copy of v fused into the
// epilogue (see RopeArgs).  qkv [M, 3*H*128], vt [M/T, H, 128, vt_keys(T)], cos_sin [T, 64].
bool gemm_mfma_qkv_rope_supported(int dtype, int M, int N, int K, int T, int H) {
  if (!gemm_mfma_supported(dtype, kEpiStore, M, N, K)) return false;
  if (N != 3 * H * 128 || H % 2 != 0 || M % T != 0) return false;
  return pick_config(kEpiQkvRope, M, N, K) >= 0;
}

// Whether the fused epilogue is the quicker way where both are open.  It excludes the tile shapes with 32-column or 80-row
// waves, which fill the chip better where they make a single round of tiles: 450 rows of 9216 columns, K = 3072, on 192 x 128 tiles and
// a rotary pass are 2 % of a forward quicker than fused on 256 x 128.  The pass moves 4 bytes per element of C at ~3.5 TB/s; a unit of
// the tile estimate is 2 K flop on one CU (~5.9 TFLOP/s).  With more rounds fused is as quick or quicker: 1281-1536 rows of 12288
// columns, K = 4096, two rounds of 192 x 256 against three of 192 x 128 and the pass, forwards 2-2.7 % quicker (3 x 437 tokens, 8 layers, 4.79
// -> 4.70 ms); 641-700 rows of 24576, K = 8192, 2 %; 1025-1140 rows of 15360, K = 5120, and 1800-1880 of 9216 within 0.5 %.
bool gemm_mfma_qkv_rope_pays(int M, int N, int K) {
  if (M <= 384) return true;
  double fused = 0, plain = 0;
  if (pick_config(kEpiQkvRope, M, N, K, &fused) < 0) return false;
  const int cfg = pick_config(kEpiStore, M, N, K, &plain);
  if (cfg < 0 || (int64_t)((M + kCfg[cfg].bm - 1) / kCfg[cfg].bm) * (N / kCfg[cfg].bn) > 256) return true;
  return fused <= plain + 2.5 * M * (double)N / K;
}

pvf_status launch_gemm_mfma_qkv_rope(pvf_ctx *ctx, hipStream_t s, const void *A, const void *W, void *qkv,
                                     void *vt, const float2 *cos_sin, int M, int N, int K, int T, int H, bool store_v,
                                     const NormArgs *na) {
  const uintptr_t al = (uintptr_t)A | (uintptr_t)W | (uintptr_t)qkv | (uintptr_t)vt;
  PVF_REQUIRE(ctx, (al & 15u) == 0, PVF_EINVAL, "gemm_mfma: operands must be 16-byte aligned");
  const int cfg = pick_config(kEpiQkvRope, M, N, K);
  PVF_REQUIRE(ctx, cfg >= 0, PVF_ESHAPE, "gemm_mfma: no tile shape with a rotary epilogue for N=%d", N);
  RopeArgs ra;
  ra.cos_sin = cos_sin; ra.vt = (bf16_t *)vt; ra.T = T; ra.Tv = vt_keys(T); ra.H = H; ra.store_v = store_v;
  PVF_REQUIRE(ctx, !na || !na->ss_in || gemm_mfma_norm_capable(cfg), PVF_ESHAPE, "gemm_mfma: tile shape %d cannot fold the norm", cfg);
  return run_cfg<kEpiQkvRope>(ctx, s, cfg, A, W, qkv, nullptr, M, N, K, ra, na ? *na : NormArgs{});
}

// QKV projection of the window rows of canvases (R rows each; windows of whole 16-key groups) with the rotary embedding and the
// key-contiguous v (vt [S][H][128][Rv]) in its epilogue: on tiles of 64 columns up to 128 rows, on the tiles of whole canvases above 384,
// where K is not divided (512 rows, cached rounds 8.65 -> 8.50 ms, 576 rows 10.66 -> 10.52).  Windows that share groups with the cache
// would have to complete them and write key by key: built, the time of the pass.
static bool window_small_tiles(int M, int N, int K) {
  const int cfg = pick_config(kEpiStore, M, N, K);
  return cfg == 6 || cfg == 12;
}
bool gemm_mfma_qkv_window_supported(int M, int N, int K) {
  if (!gemm_mfma_supported(PVF_BF16, kEpiStore, M, N, K) || N % 768 != 0) return false;
  return M > 384 ? pick_config(kEpiQkvRope, M, N, K) >= 0 && gemm_mfma_qkv_rope_pays(M, N, K) : window_small_tiles(M, N, K);
}

pvf_status launch_gemm_mfma_qkv_window(pvf_ctx *ctx, hipStream_t s, const void *A, const void *W, void *qkv, void *vt, const float2 *cos_sin,
                                       const int32_t *row_pos, int M, int N, int K, int T, int R, int Rv, int H) {
  const uintptr_t al = (uintptr_t)A | (uintptr_t)W | (uintptr_t)qkv | (uintptr_t)vt;
  PVF_REQUIRE(ctx, (al & 15u) == 0, PVF_EINVAL, "gemm_mfma: operands must be 16-byte aligned");
  PVF_REQUIRE(ctx, R > 0 && R % 16 == 0 && M % R == 0 && N == 3 * H * 128 && Rv >= R, PVF_ESHAPE, "gemm_mfma: window rows M=%d R=%d Rv=%d N=%d H=%d", M, R, Rv, N, H);
  PVF_REQUIRE(ctx, gemm_mfma_qkv_window_supported(M, N, K), PVF_ESHAPE, "gemm_mfma: window rows M=%d N=%d K=%d", M, N, K);
  RopeArgs ra{};
  ra.cos_sin = cos_sin; ra.vt = (bf16_t *)vt; ra.T = T; ra.Tv = Rv; ra.H = H; ra.row_pos = row_pos; ra.R = R;
  if (M > 384) return run_cfg<kEpiQkvRopeWin>(ctx, s, pick_config(kEpiQkvRope, M, N, K), A, W, qkv, nullptr, M, N, K, ra);
  const SplitK whole{nullptr, 0, K >= 1024};
  if (pick_config(kEpiStore, M, N, K) == 12) return run<kEpiQkvWindow, 128, 64, 64, 6, 4, 2>(ctx, s, A, W, qkv, nullptr, M, N, K, ra, whole);
  return run<kEpiQkvWindow, 64, 64, 64, 5, 2, 2>(ctx, s, A, W, qkv, nullptr, M, N, K, ra, whole);
}

bool gemm_mfma_supported(int dtype, GemmEpilogue epi, int M, int N, int K) {
  if (dtype != PVF_BF16 || M < 1 || K < 64 || K % 64 != 0) return false;
  const int64_t w_rows = (epi == kEpiSwiglu) ? 2 * (int64_t)N : N;
  if ((int64_t)M * K * 2 >= (1ll << 32) || w_rows * K * 2 >= (1ll << 32)) return false;   // 32-bit lane offsets
  return N % (epi == kEpiSwiglu ? 64 : 128) == 0;
}

// Tile shapes with room for the folded-norm exchange (every 8-wave shape).
bool gemm_mfma_norm_capable(int cfg) { return cfg >= 0 && cfg != 6 && cfg != 7 && cfg != 11 && cfg != 13; }

// Slots of row sums of squares a kEpiResidual launch writes, 256 columns each or (tiles 128 wide) 64; 0: no folded norm for
// this launch.
int gemm_mfma_norm_slots(GemmEpilogue epi, int M, int N, int K) {
  if (!gemm_mfma_supported(PVF_BF16, epi, M, N, K)) return 0;
  const int cfg = pick_config(epi, M, N, K);
  if (!gemm_mfma_norm_capable(cfg)) return 0;
  const int c = cfg == 3 || cfg >= kNumCfg ? 3 : cfg;
  return N / (kCfg[c].bn == 256 ? 256 : 64);
}

// turn: the order in which an element's k are added may depend on the launch (few rows, see kTurns).
pvf_status launch_gemm_mfma(pvf_ctx *ctx, hipStream_t s, GemmEpilogue epi, const void *A,
                            const void *W, void *C, const void *residual, int M, int N, int K, const NormArgs *na, bool turn) {
  const uintptr_t al = (uintptr_t)A | (uintptr_t)W | (uintptr_t)C | (uintptr_t)residual;
  PVF_REQUIRE(ctx, (al & 15u) == 0, PVF_EINVAL, "gemm_mfma: operands must be 16-byte aligned");
  const int cfg = pick_config(epi, M, N, K);
  PVF_REQUIRE(ctx, cfg >= 0, PVF_ESHAPE, "gemm_mfma: no tile shape for N=%d", N);
  const NormArgs nrm = na ? *na : NormArgs{};
  PVF_REQUIRE(ctx, !(nrm.ss_in || nrm.ss_out) || gemm_mfma_norm_capable(cfg), PVF_ESHAPE, "gemm_mfma: tile shape %d cannot fold the norm", cfg);
  switch (epi) {
    case kEpiStore: return run_cfg<kEpiStore>(ctx, s, cfg, A, W, C, residual, M, N, K, RopeArgs{}, NormArgs{}, turn);
    case kEpiResidual: return run_cfg<kEpiResidual>(ctx, s, cfg, A, W, C, residual, M, N, K, RopeArgs{}, nrm);
    case kEpiSwiglu: return run_cfg<kEpiSwiglu>(ctx, s, cfg, A, W, C, residual, M, N, K, RopeArgs{}, nrm, turn);
    case kEpiQkvRope: break;                     // has its own entry (launch_gemm_mfma_qkv_rope)
    case kEpiQkvWindow: case kEpiQkvRopeWin: break;      // launch_gemm_mfma_qkv_window
    case kEpiPartial: break;                     // launch_gemm_mfma_splitk
  }
  return PVF_EINVAL;
}

}  // namespace pvf
