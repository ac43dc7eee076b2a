// Grouped fp32 GEMMs (same operators as gemm_bf16.h, for the fp32 storage type): forward (NN), data gradients (NT) and
// weight gradients (TN) share one tile, 64 rows x 64 columns (GEMM-1: 64 gate and the 64 matching up columns), K never
// split, on v_mfma_f32_32x32x2_f32: fp32 operands, products and accumulators.
//
// What bounds it: the fp32 matrix pipe, 256 flop per clock and CU (154 TFLOP/s in a large library product); an MFMA of
// 4096 flop takes 64 clocks and its operands are two registers, so neither the LDS (a 16-byte and four 4-byte reads per
// four MFMAs) nor the L2 (16 bytes per clock and CU at full rate) is near its limit and the tile can stay small, which
// is what the small layers need.  Four waves, 32 x 32 each (GEMM-1: twice), K step 16, two LDS stages and two more
// steps in registers: a load has about two steps (1000 clocks and more) to arrive, at one workgroup per CU as in the
// single launch; the serialized launches run four per CU, whose waves hide each other's barriers.
// Both operands go through LDS, either k-contiguous (rows of 16 + 4 floats: the 16-byte fragment reads of 16 lanes
// cover all banks) or x-contiguous (rows of 64 + 8 floats: the two half-waves read rows four apart from different
// banks).  A lane's fragment of eight k is k = 4 * (lane / 32) .. + 3, one MFMA per component: the pairing of k with
// the MFMA's two k slots is the same for both operands, so it only fixes the order of the sum.
// Result layout: lane = column, register r = row 8 * (r / 4) + 4 * (lane / 32) + r % 4: a store writes whole
// 128-byte lines of two rows.
// Measured, T = 1500, H = 1024, I = 704, 16 experts, k = 4 (25.9 GFLOP forward, 51.9 backward), against 64 x 64 tiles with
// 4 x 4 outputs per thread on the vector ALU: GEMM-1 418 -> 190 us (91 TFLOP/s), GEMM-2 173 -> 97, act_grad 277 -> 112,
// gate_grad 521 -> 185, the two weight gradients 371 -> 144 each; error against 64 bits unchanged (1.0e-6).  The matrix
// pipe is 83 % busy on a busy CU (GEMM-1); the rest is the last round: 1056 tiles on 256 CUs are 4.1 per CU.
#pragma once
#include "common.h"
#include "gemm_bf16.h"  // GemmEpilogue, xcd_spread_tile

namespace moe {

constexpr int kFBM = 64, kFBN = 64, kFBK = 16;
constexpr int kFKcLd = kFBK + 4;                  // k-contiguous stage: floats per row
constexpr int kFXcLd = kFBN + 8;                  // x-contiguous stage: floats per k
constexpr int kFStage = kFBM * kFKcLd;            // floats per operand stage (1280 >= 16 * 72)
static_assert(kFStage >= kFBK * kFXcLd, "stage size");
constexpr int kFLdsFloats1 = 2 * 2 * kFStage;     // two stages of two operands (20 KB)
constexpr int kFLdsFloats2 = 2 * 3 * kFStage;     // two weight column blocks (30 KB)

struct GemmParamsF32 {
  const float* A;   // [rows, lda]
  const float* B;   // per expert [K, ldb]
  float* C;         // [rows, ldc]
  float* C2;        // SwiGLU only: optional pre-activation [rows, 2N]
  long strideB;
  int K, N;         // N = output columns (SwiGLU: I)
  int lda, ldb, ldc;
  int n_ntiles;     // N / 64
  TileMap tiles;
};

typedef __attribute__((address_space(3))) float* lds_f32_ptr;
typedef __attribute__((address_space(3))) f32x4* lds_f32x4_ptr;

// acc[h] += A * B_h over n_steps K steps of 16 (rounded up to an even count) for this wave's 32 x 32 block (wm, wn).
// A_KC / B_KC: operand k-contiguous (a thread fetches row tid / 4, k = tid % 4 * 4 .. + 3) or x-contiguous (k = tid / 16,
// columns tid % 16 * 4 .. + 3); a_ptr / b_ptr: this thread's 16 bytes of step 0, a_k / b_k: floats from one k to the next,
// b_half: floats between the column blocks.  K_TAIL (both operands x-contiguous): K need not be a multiple of 16; what lies
// past it is zero in both operands.  ACTIVE: the wave has rows (its accumulators stay out of any branch: a branch inside
// the loop made the compiler copy them between the register files on every step).
// Loads are unconditional (past the last step they repeat it), so that a wait names exactly the older of the two steps
// that are under way.
template <bool A_KC, bool B_KC, int NB, bool K_TAIL, bool ACTIVE>
__device__ __forceinline__ void gemm_core_f32(f32x16 (&acc)[NB], const float* a_ptr, long a_k, const float* b_ptr, long b_k,
                                              long b_half, int K, float* smem) {
  static_assert(!K_TAIL || (!A_KC && !B_KC), "ragged K: x-contiguous operands");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, lh = lane >> 5;
  const int n_steps = (K + kFBK - 1) / kFBK;
  const int kt = tid >> 4;                             // K_TAIL: this thread's k inside a step
  const lds_f32_ptr lds = (lds_f32_ptr)smem;
  constexpr int kStages = (1 + NB) * kFStage;          // floats of one stage of all operands
  const int a_st = A_KC ? (tid >> 2) * kFKcLd + (tid & 3) * 4 : kt * kFXcLd + (tid & 15) * 4;
  const int b_st = B_KC ? (tid >> 2) * kFKcLd + (tid & 3) * 4 : kt * kFXcLd + (tid & 15) * 4;
  const int a_rd = A_KC ? (wm * 32 + l32) * kFKcLd + lh * 4 : lh * 4 * kFXcLd + wm * 32 + l32;
  const int b_rd = B_KC ? (wn * 32 + l32) * kFKcLd + lh * 4 : lh * 4 * kFXcLd + wn * 32 + l32;
  struct Regs { f32x4 a, b[NB]; };
  auto load = [&](Regs& r, int s) __attribute__((always_inline)) {
    const long k = K_TAIL ? min(s * kFBK + kt, K - 1) - kt : min(s, n_steps - 1) * kFBK;
    r.a = *reinterpret_cast<const f32x4*>(a_ptr + k * a_k);
#pragma unroll
    for (int h = 0; h < NB; ++h) r.b[h] = *reinterpret_cast<const f32x4*>(b_ptr + k * b_k + h * b_half);
  };
  auto stage = [&](const Regs& r, int s, int buf) __attribute__((always_inline)) {
    const lds_f32_ptr st = lds + buf * kStages;
    const bool in = !K_TAIL || s * kFBK + kt < K;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    *(lds_f32x4_ptr)(st + a_st) = in ? r.a : z;
#pragma unroll
    for (int h = 0; h < NB; ++h) *(lds_f32x4_ptr)(st + (1 + h) * kFStage + b_st) = in ? r.b[h] : z;
  };
  auto compute = [&](int buf) __attribute__((always_inline)) {
    if (!ACTIVE) return;
    const lds_f32_ptr as = lds + buf * kStages + a_rd;
    f32x4 a[2], b[2][NB];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (A_KC) a[q] = *(lds_f32x4_ptr)(as + q * 8);
      else {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[q][i] = as[(q * 8 + i) * kFXcLd];
      }
#pragma unroll
      for (int h = 0; h < NB; ++h) {
        const lds_f32_ptr bs = lds + buf * kStages + (1 + h) * kFStage + b_rd;
        if (B_KC) b[q][h] = *(lds_f32x4_ptr)(bs + q * 8);
        else {
#pragma unroll
          for (int i = 0; i < 4; ++i) b[q][h][i] = bs[(q * 8 + i) * kFXcLd];
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);                 // all reads of the step ahead of its first MFMA: one LDS latency per step
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < NB; ++h) acc[h] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][i], b[q][h][i], acc[h], 0, 0, 0);
  };
  if (n_steps <= 0) return;
  Regs r0, r1;
  load(r0, 0);
  load(r1, 1);
  stage(r0, 0, 0);
  if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
  load(r0, 2);
  __syncthreads();
  for (int s = 0; s < n_steps; s += 2) {   // an odd count (ragged K only) ends with a step of zeros
    compute(0);
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);   // the zeroing of one step must not be moved ahead of the other's wait
    stage(r1, s + 1, 1);
    load(r1, s + 3);
    __syncthreads();
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
    compute(1);
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
    stage(r0, s + 2, 0);
    load(r0, s + 4);
    __syncthreads();                       // also: LDS free for the next tile
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
  }
}

template <bool A_KC, bool B_KC, int NB>
__device__ __forceinline__ void gemm_rows_f32(f32x16 (&acc)[NB], const float* a_ptr, long a_k, const float* b_ptr, long b_k,
                                              long b_half, int K, bool active, float* smem) {
  if (active) gemm_core_f32<A_KC, B_KC, NB, false, true>(acc, a_ptr, a_k, b_ptr, b_k, b_half, K, smem);
  else gemm_core_f32<A_KC, B_KC, NB, false, false>(acc, a_ptr, a_k, b_ptr, b_k, b_half, K, smem);
}

// Rows of a wave's block in the order of the result registers.
__device__ __forceinline__ int f32_acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

template <int EPI>
__device__ __forceinline__ void gemm_tile_f32(const GemmParamsF32& p, int mtile, int ntile, float* smem) {
  constexpr int NB = (EPI == kEpiSwiglu) ? 2 : 1;   // weight column blocks per tile (gate, up)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int e = p.tiles.expert[mtile];
  const int row0 = p.tiles.row0[mtile];
  const int rows = p.tiles.rows[mtile];
  if (rows <= 0) return;   // the empty half of a pair slot (block-uniform)
  const int n0 = ntile * kFBN;
  f32x16 acc[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[h][r] = 0.f;
  gemm_rows_f32<true, false, NB>(acc, p.A + (size_t)(row0 + min(tid >> 2, rows - 1)) * p.lda + (tid & 3) * 4, 1,
                                 p.B + (size_t)e * p.strideB + (size_t)(tid >> 4) * p.ldb + n0 + (tid & 15) * 4, p.ldb, p.N, p.K,
                                 wm * 32 < rows, smem);
  const int c = n0 + wn * 32 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = wm * 32 + f32_acc_row(r, lane);
    if (m >= rows) continue;
    const size_t grow = (size_t)(row0 + m);
    if (EPI == kEpiSwiglu) {
      const float g = acc[0][r], u = acc[NB - 1][r];
      p.C[grow * p.ldc + c] = g * sigmoidf_(g) * u;
      if (p.C2) {
        p.C2[grow * (size_t)(2 * p.N) + c] = g;
        p.C2[grow * (size_t)(2 * p.N) + p.N + c] = u;
      }
    } else {
      p.C[grow * p.ldc + c] = acc[0][r];
    }
  }
}

template <int EPI>
__global__ __launch_bounds__(256) void grouped_gemm_f32_kernel(GemmParamsF32 p) {
  __shared__ __attribute__((aligned(16))) float smem[EPI == kEpiSwiglu ? kFLdsFloats2 : kFLdsFloats1];
  const int total = p.tiles.meta[kMetaMTiles] * p.n_ntiles;
  const int G = gridDim.x;
  for (int it = 0; it * G < total; ++it) {
    const int tile = xcd_spread_tile(it, blockIdx.x, G, total);
    if (tile < 0) continue;
    gemm_tile_f32<EPI>(p, tile / p.n_ntiles, tile % p.n_ntiles, smem);
  }
}

}  // namespace moe
