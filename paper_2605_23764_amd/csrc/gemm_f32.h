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
// pipe is 83 % busy on a busy CU (GEMM-1).  With quarter tiles for the last round (1111 tiles on 256 CUs are 4.3 per CU):
// GEMM-1 190 -> 178, act_grad 114 -> 102; where a whole launch has few tiles more: T = 256, H = 256, I = 128, 8 experts, a
// training step 72.7 -> 52 (GEMM-1 14.4 -> 7.1, act_grad 14.4 -> 7.2, gate_grad 8.3 -> 5.3); T = 300, H = 512, I = 448, 10 of 16
// experts 116.7 -> 91.5; T = 20, H = 2048, I = 1408, forward 168 -> 150.  Same bits.
// No gain from deeper prefetch (four steps in registers), operand fragments read a step ahead, or wave priorities by what
// a workgroup has left.
#pragma once
#include "common.h"
#include "gemm_bf16.h"  // GemmEpilogue, xcd_spread_tile

namespace moe {

constexpr int kFBM = 64, kFBN = 64, kFBK = 16;
constexpr int kFKcLd = kFBK + 4;                  // k-contiguous stage: floats per row
constexpr int kFXcLd = kFBN + 8;                  // x-contiguous stage: floats per k
constexpr int kFStage = kFBM * kFKcLd;            // floats per operand stage (1280 >= 16 * 72)
static_assert(kFStage >= kFBK * kFXcLd, "stage size");
constexpr int kFQK = 32, kFQLd = 32 + 4;          // a quarter tile's K step; floats per row (either orientation)
constexpr int kFQFixed = 64;                      // what a tile of either size costs beside its K loop, in k of a quarter
constexpr int kFQStage = 32 * kFQLd;
static_assert(kFQStage <= kFStage, "a quarter's stages fit where a tile's do");
constexpr int kFLdsFloats1 = 2 * 2 * kFStage;     // two stages of two operands (20 KB)
constexpr int kFLdsFloats2 = 2 * 3 * kFStage;     // two weight column blocks (30 KB)

constexpr int kFSLd = 64 + 4;                     // a strip's weight stage: floats per k
// LDS of a serialized launch: two stages of tiles or of strips (22 KB; two weight column blocks 39 KB, four workgroups a CU)
constexpr int f32_lds_floats(int nb) { return 2 * (16 * kFQLd + nb * kFQK * kFSLd); }
static_assert(f32_lds_floats(1) >= kFLdsFloats1 && f32_lds_floats(2) >= kFLdsFloats2 && 4 * 4 * f32_lds_floats(2) <= 160 * 1024, "LDS budget");

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
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f32x2* lds_f32x2_ptr;

// The same address, of which the compiler knows nothing: it stays in its register.
__device__ __forceinline__ lds_f32_ptr lds_pinned(lds_f32_ptr p) {
  uint32_t a = (uint32_t)(uintptr_t)p;
  asm volatile("" : "+v"(a));
  return (lds_f32_ptr)(uintptr_t)a;
}

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
  // Where an x-contiguous operand's reads of eight k start, per stage.  Opaque, or in the long body of the single launch the
  // compiler adds them up again on every step, between the barrier and the reads (GEMM-1: 112 instructions per two steps instead
  // of 100; single launch, H = 2048, I = 1408, 16 of 64 experts, 90 rows per expert 413 -> 403 us, 250 rows 850 -> 832; H = 1024,
  // I = 704, 16 experts, 375 rows 385 -> 378); the other launches have the same loops either way.
  lds_f32_ptr a_at[2][2], b_at[2][NB][2];
#pragma unroll
  for (int buf = 0; buf < 2; ++buf)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (!A_KC) a_at[buf][q] = lds_pinned(lds + buf * kStages + a_rd + q * 8 * kFXcLd);
#pragma unroll
      for (int h = 0; h < NB; ++h)
        if (!B_KC) b_at[buf][h][q] = lds_pinned(lds + buf * kStages + (1 + h) * kFStage + b_rd + q * 8 * kFXcLd);
    }
  auto compute = [&](int buf) __attribute__((always_inline)) {
    if (!ACTIVE) return;
    const lds_f32_ptr as = lds + buf * kStages + a_rd;
    f32x4 a[2], b[2][NB];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (A_KC) a[q] = *(lds_f32x4_ptr)(as + q * 8);
      else {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[q][i] = a_at[buf][q][i * kFXcLd];
      }
#pragma unroll
      for (int h = 0; h < NB; ++h) {
        if (B_KC) b[q][h] = *(lds_f32x4_ptr)(lds + buf * kStages + (1 + h) * kFStage + b_rd + q * 8);
        else {
#pragma unroll
          for (int i = 0; i < 4; ++i) b[q][h][i] = b_at[buf][h][q][i * kFXcLd];
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

// A quarter of a tile, 32 x 32, for launches and last rounds with too few tiles: wave (wm, wn) owns a 16 x 16 block (GEMM-1:
// twice) on v_mfma_f32_16x16x4_f32, K step 32, two LDS stages and four more steps in registers.  Both MFMA shapes add one
// product after the other, in the order of their k slots (bit for bit the chain of fmaf: 204 800 random results), so with the
// slots 0 4 1 5, then 2 6 3 7 of every eight k the quarter gives the same bits as the whole tile, whose slots are 0 4, 1 5,
// 2 6, 3 7.  The k-contiguous stage keeps a lane group's eight k of a step together (group g = lane / 16 holds k = 4 * (g & 1)
// + g / 2, + 2 of every eight): rows of 4 x 8 + 4 floats, read as two 16-byte fragments without conflicts.
template <bool A_KC, bool B_KC, int NB, bool K_TAIL>
__device__ __forceinline__ void gemm_core_f32_quarter(f32x4 (&acc)[NB], const float* a_ptr, long a_k, const float* b_ptr, long b_k,
                                                      long b_half, int K, float* smem) {
  static_assert(!K_TAIL || (!A_KC && !B_KC), "ragged K: x-contiguous operands");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;
  const int n_steps = (K + kFQK - 1) / kFQK;
  const int kt = tid >> 3;                             // K_TAIL: this thread's k inside a step
  const lds_f32_ptr lds = (lds_f32_ptr)smem;
  constexpr int kStages = (1 + NB) * kFQStage;
  constexpr int kAhead = NB == 1 ? 4 : 2;              // steps under way (GEMM-1: two, or fewer than four workgroups fit a CU)
  const int kc_st = (tid >> 3) * kFQLd + (tid & 1) * 8 + ((tid & 7) >> 1) * 2, xc_st = kt * kFQLd + (tid & 7) * 4;
  const int k0 = (lg & 1) * 4 + (lg >> 1);
  const int a_rd = A_KC ? (wm * 16 + l16) * kFQLd + lg * 8 : k0 * kFQLd + wm * 16 + l16;
  const int b_rd = B_KC ? (wn * 16 + l16) * kFQLd + lg * 8 : k0 * kFQLd + wn * 16 + l16;
  struct Regs { f32x4 a, b[NB]; };
  auto load = [&](Regs& r, int s) __attribute__((always_inline)) {
    const long k = K_TAIL ? min(s * kFQK + kt, K - 1) - kt : min(s, n_steps - 1) * kFQK;
    r.a = *reinterpret_cast<const f32x4*>(a_ptr + k * a_k);
#pragma unroll
    for (int h = 0; h < NB; ++h) r.b[h] = *reinterpret_cast<const f32x4*>(b_ptr + k * b_k + h * b_half);
  };
  auto put = [&](lds_f32_ptr st, const f32x4& v, bool kc) __attribute__((always_inline)) {
    if (kc) {
      *(lds_f32x2_ptr)(st + kc_st) = f32x2{v[0], v[2]};
      *(lds_f32x2_ptr)(st + kc_st + 16) = f32x2{v[1], v[3]};
    } else {
      *(lds_f32x4_ptr)(st + xc_st) = v;
    }
  };
  auto stage = [&](const Regs& r, int s, int buf) __attribute__((always_inline)) {
    const lds_f32_ptr st = lds + buf * kStages;
    const bool in = !K_TAIL || s * kFQK + kt < K;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    put(st, in ? r.a : z, A_KC);
#pragma unroll
    for (int h = 0; h < NB; ++h) put(st + (1 + h) * kFQStage, in ? r.b[h] : z, B_KC);
  };
  auto fragment = [&](float (&f)[8], lds_f32_ptr st, bool kc) __attribute__((always_inline)) {
    if (kc) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4 v = *(lds_f32x4_ptr)(st + q * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[q * 4 + i] = v[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = st[((i >> 1) * 8 + (i & 1) * 2) * kFQLd];
    }
  };
  auto step = [&](Regs& r, int s, int buf) __attribute__((always_inline)) {
    const lds_f32_ptr st = lds + buf * kStages;
    float a[8], b[NB][8];
    fragment(a, st + a_rd, A_KC);
#pragma unroll
    for (int h = 0; h < NB; ++h) fragment(b[h], st + (1 + h) * kFQStage + b_rd, B_KC);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < NB; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[h][i], acc[h], 0, 0, 0);
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);     // the zeroing of one step must not be moved ahead of the other's wait
    stage(r, s + 1, buf ^ 1);
    load(r, s + 1 + kAhead);
    __syncthreads();                                   // at the last step also: LDS free for the next tile
    if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
  };
  if (n_steps <= 0) return;
  Regs r[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) load(r[i], i);
  stage(r[0], 0, 0);
  if (K_TAIL) __builtin_amdgcn_sched_barrier(0);
  load(r[0], kAhead);
  __syncthreads();
  for (int s = 0; s < n_steps; s += kAhead) {          // an odd count (ragged K only) ends with a step of zeros
    step(r[1], s, 0);
    step(r[2 % kAhead], s + 1, 1);
    if constexpr (kAhead == 4) {
      if (s + 2 >= n_steps) break;
      step(r[3], s + 2, 0);
      step(r[0], s + 3, 1);
    }
  }
}

// A strip, 16 rows x 64 columns, for launches whose experts have at most 16 rows each: wave w owns columns 16 w .. + 15 (GEMM-1:
// of the gate and of the up block) and nothing is multiplied for rows that are not there, K step 32.  Such a launch reads
// weights: 256-byte pieces, AHEAD steps of 8 KB (GEMM-1: 16) under way per workgroup.  Forward layout only; the same chain of
// sums as the other tiles.  Against quarters (whose second 16 rows do not exist here, and which read 128-byte pieces): forward of
// T = 20, H = 2048, I = 1408, 16 of 64 experts 145 -> 95 us (554 MB of weights where all have rows, 78 us at 7.1 TB/s), T = 100 180 -> 118;
// T = 30, H = 1024, I = 704, 16 experts 61.6 -> 42; T = 8, 64 experts 115 -> 75.  With two quarters per tile up to 32 rows: T = 64
// 62.6 -> 52.7, a training step of T = 64, H = 512, I = 448, 10 of 16 experts 75 -> 63.5.
template <int NB, int AHEAD>
__device__ __forceinline__ void gemm_core_f32_strip(f32x4 (&acc)[NB], const float* a_ptr, const float* b_ptr, long b_k, long b_half,
                                                    int K, float* smem) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int n_steps = K / kFQK;                        // even: K is a multiple of 64
  const lds_f32_ptr lds = (lds_f32_ptr)smem;
  constexpr int kAStage = 16 * kFQLd, kBStage = kFQK * kFSLd, kStages = kAStage + NB * kBStage;
  static_assert(2 * kStages <= f32_lds_floats(NB), "LDS budget");
  const bool has_a = wave < 2;                         // 128 threads fetch the 16 rows
  const int a_st = (tid >> 3) * kFQLd + (tid & 1) * 8 + ((tid & 7) >> 1) * 2;
  const int b_st = kAStage + (tid >> 4) * kFSLd + (tid & 15) * 4;
  const int k0 = (lg & 1) * 4 + (lg >> 1);
  const int a_rd = l16 * kFQLd + lg * 8, b_rd = kAStage + k0 * kFSLd + wave * 16 + l16;
  struct Regs { f32x4 a, b[NB][2]; } r[AHEAD];
  auto load = [&](Regs& q, int s) __attribute__((always_inline)) {
    const long k = (long)min(s, n_steps - 1) * kFQK;
    q.a = *reinterpret_cast<const f32x4*>(a_ptr + k);
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        q.b[h][i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(b_ptr + (k + 16 * i) * b_k + h * b_half));
  };
  auto stage = [&](const Regs& q, int buf) __attribute__((always_inline)) {
    const lds_f32_ptr st = lds + buf * kStages;
    if (has_a) {
      *(lds_f32x2_ptr)(st + a_st) = f32x2{q.a[0], q.a[2]};
      *(lds_f32x2_ptr)(st + a_st + 16) = f32x2{q.a[1], q.a[3]};
    }
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) *(lds_f32x4_ptr)(st + b_st + h * kBStage + i * 16 * kFSLd) = q.b[h][i];
  };
  auto step = [&](Regs& q, int s, int buf) __attribute__((always_inline)) {
    const lds_f32_ptr st = lds + buf * kStages;
    f32x4 a[2];
    float b[NB][8];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *(lds_f32x4_ptr)(st + a_rd + i * 4);
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) b[h][i] = st[b_rd + h * kBStage + ((i >> 1) * 8 + (i & 1) * 2) * kFSLd];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < NB; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i >> 2][i & 3], b[h][i], acc[h], 0, 0, 0);
    stage(q, buf ^ 1);
    load(q, s + 1 + AHEAD);
    __syncthreads();                                   // at the last step also: LDS free for the next tile
  };
  if (n_steps <= 0) return;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) load(r[i], i);
  stage(r[0], 0);
  load(r[0], AHEAD);
  __syncthreads();
  for (int s = 0; s < n_steps; s += AHEAD) {
    step(r[1], s, 0);
    step(r[2 % AHEAD], s + 1, 1);
    if constexpr (AHEAD == 4) {
      if (s + 2 >= n_steps) break;
      step(r[3], s + 2, 0);
      step(r[0], s + 3, 1);
    }
  }
}

// Tiles of a launch of G workgroups, four to a CU: whole tiles in full sweeps, the rest as quarters where that shortens the
// launch.  The fullest CU decides: ceil(4 rem / G) whole tiles or ceil(16 rem / G) quarters (half_rows: no tile has more than 32
// rows, two quarters each).  A quarter fetches twice the
// operand bytes per product, an eighth on its time; kFQFixed: a weight gradient over 60 rows per expert (560 tiles) is faster
// whole (a step of T = 300 91.9 us against 93.1), GEMMs of K = 1024 are not (forward of T = 600, 528 tiles: 161 -> 147).
template <typename Whole, typename Quarter>
__device__ __forceinline__ void f32_sweeps(int b, int total, int K, bool half_rows, Whole&& whole, Quarter&& quarter) {
  const int G = gridDim.x, rem = total % G, nq = half_rows ? 2 : 4;
  const bool split = (4 * nq * rem + G - 1) / G * (9 * K + 8 * kFQFixed) < (4 * rem + G - 1) / G * (32 * K + 8 * kFQFixed);
  const int n_whole = split ? total - rem : total;
  for (int it = 0; it * G < n_whole; ++it) {
    const int tile = xcd_spread_tile(it, b, G, n_whole);
    if (tile >= 0) whole(tile);
  }
  if (!split) return;
  for (int it = 0; it * G < nq * rem; ++it) {
    const int i = xcd_spread_tile(it, b, G, nq * rem);
    if (i >= 0) quarter(n_whole + (half_rows ? i >> 1 : i >> 2), half_rows ? 0 : (i >> 1) & 1, i & 1);
  }
}

// Rows of a wave's block in the order of the result registers.
__device__ __forceinline__ int f32_acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// One result: v, for SwiGLU the pre-activations (v, u).
template <int EPI>
__device__ __forceinline__ void store_f32(const GemmParamsF32& p, size_t grow, int c, float v, float u) {
  if (EPI == kEpiSwiglu) {
    p.C[grow * p.ldc + c] = v * sigmoidf_(v) * u;
    if (p.C2) {
      p.C2[grow * (size_t)(2 * p.N) + c] = v;
      p.C2[grow * (size_t)(2 * p.N) + p.N + c] = u;
    }
  } else {
    p.C[grow * p.ldc + c] = v;
  }
}

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
    if (m < rows) store_f32<EPI>(p, (size_t)(row0 + m), c, acc[0][r], acc[NB - 1][r]);
  }
}

// Quarter (qm, qn) of the same tile.
template <int EPI>
__device__ __forceinline__ void gemm_quarter_f32(const GemmParamsF32& p, int mtile, int ntile, int qm, int qn, float* smem) {
  constexpr int NB = (EPI == kEpiSwiglu) ? 2 : 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int e = p.tiles.expert[mtile];
  const int row0 = p.tiles.row0[mtile] + qm * 32;
  const int rows = p.tiles.rows[mtile] - qm * 32;
  if (rows <= 0) return;
  const int n0 = ntile * kFBN + qn * 32;
  f32x4 acc[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[h][r] = 0.f;
  gemm_core_f32_quarter<true, false, NB, false>(acc, p.A + (size_t)(row0 + min(tid >> 3, rows - 1)) * p.lda + (tid & 7) * 4, 1,
                                                p.B + (size_t)e * p.strideB + (size_t)(tid >> 3) * p.ldb + n0 + (tid & 7) * 4,
                                                p.ldb, p.N, p.K, smem);
  const int c = n0 + wn * 16 + (lane & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = wm * 16 + 4 * (lane >> 4) + r;
    if (m < rows) store_f32<EPI>(p, (size_t)(row0 + m), c, acc[0][r], acc[NB - 1][r]);
  }
}

// The same tile of an expert with at most 16 rows.
// AHEAD: steps under way, two where four workgroups share a CU (four are no faster there and take too many registers).
template <int EPI, int AHEAD = 2>
__device__ __forceinline__ void gemm_strip_f32(const GemmParamsF32& p, int mtile, int ntile, float* smem) {
  constexpr int NB = (EPI == kEpiSwiglu) ? 2 : 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int e = p.tiles.expert[mtile], row0 = p.tiles.row0[mtile], rows = p.tiles.rows[mtile];
  if (rows <= 0) return;
  const int n0 = ntile * kFBN;
  f32x4 acc[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[h][r] = 0.f;
  gemm_core_f32_strip<NB, AHEAD>(acc, p.A + (size_t)(row0 + min((tid >> 3) & 15, rows - 1)) * p.lda + (tid & 7) * 4,
                          p.B + (size_t)e * p.strideB + (size_t)(tid >> 4) * p.ldb + n0 + (tid & 15) * 4, p.ldb, p.N, p.K, smem);
  const int c = n0 + (tid >> 6) * 16 + (lane & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = 4 * (lane >> 4) + r;
    if (m < rows) store_f32<EPI>(p, (size_t)(row0 + m), c, acc[0][r], acc[NB - 1][r]);
  }
}

// A tile as a task of the single launch, whose one workgroup per CU has registers for four steps under way.  Tiles of at most 16
// rows as strips: T = 20, H = 2048, I = 1408, 16 of 64 experts, single launch 219 -> 141 us, T = 1 86 -> 58; T = 8, H = 1024, I = 704,
// 64 experts 173 -> 130; 128 rows per expert, whose last tile is often a strip, 551 -> 487.  More rows don't lose by the longer code
// with the LDS addresses of the tile pinned (gemm_core_f32): 375 rows 383 -> 378, without that 385.  Of 35 calls of 1..375 rows
// one is slower than whole tiles: skewed routing of T = 192 over 16 experts, 137 -> 139 (of T = 128 157 -> 143).
template <int EPI>
__device__ __forceinline__ void gemm_task_f32(const GemmParamsF32& p, int mtile, int ntile, float* smem) {
  if (__builtin_amdgcn_readfirstlane(p.tiles.rows[mtile]) <= 16) gemm_strip_f32<EPI, 4>(p, mtile, ntile, smem);
  else gemm_tile_f32<EPI>(p, mtile, ntile, smem);
}

template <int EPI>
__global__ __launch_bounds__(256, EPI == kEpiSwiglu ? 4 : 1) void grouped_gemm_f32_kernel(GemmParamsF32 p) {
  __shared__ __attribute__((aligned(16))) float smem[f32_lds_floats(EPI == kEpiSwiglu ? 2 : 1)];
  const int total = p.tiles.meta[kMetaMTiles] * p.n_ntiles;
  const int max_rows = p.tiles.meta[kMetaMaxRows], G = gridDim.x;
  // strips where two quarters per tile would not find a CU each (T = 4, H = 2048, I = 1408, about four experts with rows: 51 us a
  // layer with quarters, 59 with strips; T = 20, 12 experts: 145 and 95)
  if (max_rows <= 16 && 8 * total > G) {
    for (int it = 0; it * G < total; ++it) {
      const int t = xcd_spread_tile(it, blockIdx.x, G, total);
      if (t >= 0) gemm_strip_f32<EPI>(p, t / p.n_ntiles, t % p.n_ntiles, smem);
    }
    return;
  }
  f32_sweeps(blockIdx.x, total, p.K, max_rows <= 32,
             [&](int t) __attribute__((always_inline)) { gemm_tile_f32<EPI>(p, t / p.n_ntiles, t % p.n_ntiles, smem); },
             [&](int t, int qm, int qn) __attribute__((always_inline)) {
               gemm_quarter_f32<EPI>(p, t / p.n_ntiles, t % p.n_ntiles, qm, qn, smem);
             });
}

}  // namespace moe
