// Grouped bf16 GEMMs for a few rows per expert (serving batches, small training batches): the weight stream.
//
// With at most 64 rows per expert a weight element meets one or two MFMA row blocks, so the launch is a read of the
// weights at HBM rate and nothing else (up to 128 rows, where a launch is a single round: stream_takes); the tile of
// gemm_bf16.h (256 weight columns, 64 KB of weights under way per CU) then has too few work items to fill the chip evenly
// (T = 1 at H = 2048, I = 1408: 44 items on four of the eight dies) and too little in flight.  Here
//   * an item is some weight columns of one expert over the whole K (never split: results are the same bits as the other
//     kernel's, whose MFMAs sum in the same order), dealt evenly to all workgroups.  Three widths (stream_rule.h has the rule):
//       columns                a stage holds (weights)   ring: up to 16 / 32 / 64 / 128 rows   weights under way
//       256 (GEMM-1 only)      64 k x 256 = 32 KB        4 / 4 / 3 / -  stages                 96 .. 64 KB
//       128                    64 k x 128 = 16 KB        7 / 7 / 6 / 4                         96 .. 48 KB
//       64                     128 k x 64 = 16 KB        7 / 6 / 4 / 3                         96 .. 32 KB
//   * a workgroup runs its items as ONE stream of such stages through the ring in LDS; the next item's first stages are
//     requested while the last ones of this item are multiplied, so nothing drains between items;
//   * activation rows ride along in the same stage (4 to 32 KB, from the L2), gathered through the permutation if need be;
//   * one barrier per stage; each of the four waves multiplies one 32-column block (256 columns: two; 64 columns: two of the
//     waves one each, above 32 rows two waves a block, half of the rows each).  For SwiGLU a block is 16 gate and the 16
//     matching up columns: both meet in one lane's accumulators.
// Results are written straight from the accumulators (8 bytes per lane): they are a thousandth of the bytes read.
// The weights are read non-temporally (each line once, by one workgroup; 64 columns: not, two items share a line): 5 to 9 %
// of a launch.
// What bounds it: the rate at which HBM serves short pieces of rows 4..14 KB apart: 256 bytes, 128 where a SwiGLU item of 128
// columns reads 64 gate and 64 up columns.  A loop that only loads pieces of 256 bytes reaches 6.2 TB/s (5.7 without the
// non-temporal hint; 128 bytes 5.1), 1 KB pieces 6.3..6.7, one linear stream 7.1; with the MFMAs taken out the launch is no
// faster, without the activation loads 2 %.
// Measured, layer (routing and Combine included), against the tiles of gemm_bf16.h: H = 7168, I = 2048, 32 of 256 experts,
// k = 8: T = 4 168 -> 101 us, T = 32 428 -> 354 (328 with the rest of a round as 128 columns: stream_wide), T = 256 524 -> 461,
// T = 1000 548 -> 505; H = 2048, I = 1408, 16 experts, k = 4: T = 1 60 -> 38.5, T = 8 74 -> 62, T = 64 76 -> 67.  Above 64 rows the activations' share of a stage grows past a
// third and the other kernel's 256 rows per weight fetch win, unless its tiles leave CUs idle.
#pragma once
#include "gemm_bf16.h"

namespace moe {

constexpr int kStreamRing = 144 * 1024;              // LDS of the stages
constexpr int kStreamGather = 2048;                  // token indices kept in LDS (rows beyond are looked up in memory)

// CW weight columns per item; AL activation lines (8 rows x 64 k) per wave and stage.
template <int CW, int AL>
struct StreamShape {
  static constexpr int kKB = CW == 64 ? 128 : 64;                // k per stage
  static constexpr int kRows = (CW == 64 ? 16 : 32) * AL;        // activation rows a stage holds
  static constexpr int kMT = kRows > 32 ? kRows / 32 : 1;        // 32-row blocks
  static constexpr int kWaveRows = CW == 64 && kMT > 1 ? 2 : 1;  // 64 columns: the waves share two column blocks and split the rows
  static constexpr int kMTW = kMT / kWaveRows;                   // row blocks per wave
  static constexpr int kNB = CW == 256 ? 2 : 1;                  // 32-column blocks per wave
  static constexpr int kBLoads = CW == 256 ? 8 : 4;              // weight lines per wave and stage
  static constexpr int kALine0 = 4 * kBLoads;                    // the stage's activation lines follow its weight lines
  static constexpr int kStage = (kALine0 + 4 * AL) * kLine;
  static constexpr int kDepth = kStreamRing / kStage;
  static constexpr int kLoads = kBLoads + AL;                    // wave-wide loads per wave and stage
};

constexpr int kStreamTables = kStreamRing;           // LDS offset of the tables, behind the ring
constexpr int kStreamGatherOff = kStreamTables + 3 * kMaxE * 4;
constexpr int kStreamBox = kStreamGatherOff + kStreamGather * 4;   // three words of the single launch (stream_layer.h)
static_assert(kStreamBox + 12 <= kGemmLdsBytes, "LDS budget");

// Who runs a stream: a launch of its own; or both GEMMs of a layer one after the other in the single launch (stream_layer.h),
// whose results are stored through to memory and whose second stream starts with the weights, before the activations are there.
enum StreamRole { kStreamAlone = 0, kStreamFirst = 1, kStreamSecond = 2 };

typedef __attribute__((address_space(3))) int32_t* lds_i32_ptr;
// 8 bytes of a result; THROUGH: as store_through does.
template <bool THROUGH>
__device__ __forceinline__ void store8(__bf16* dst, u32x2 v) {
  if constexpr (THROUGH) asm volatile("global_store_dwordx2 %0, %1, off sc1\n\ts_nop 1" : : "v"(dst), "v"(v) : "memory");
  else *reinterpret_cast<u32x2*>(dst) = v;
}

// Waits until at most `stages` stages requested after the wanted one are under way (fewer near the end of the stream).
template <int LPS, int MOST>
__device__ __forceinline__ void stream_wait(int stages) {
  if constexpr (MOST == 0) {
    wait_vmcnt<0>();
  } else {
    if (stages >= MOST) wait_vmcnt<LPS * MOST>();
    else stream_wait<LPS, MOST - 1>(stages);
  }
}

// Items id0 .. id1 - 1 (expert by expert among those with rows, then by columns), the share of workgroup b.  kStreamSecond: ready()
// waits until the activations may be read; false, it has given up, and nothing is stored.
template <int LAY, int EPI, int CW, int AL, int ROLE, typename Ready>
__device__ __forceinline__ void stream_items(const GemmParams& p, int id0, int id1, int b, char* smem, Ready&& ready) {
  typedef StreamShape<CW, AL> S;
  constexpr int kOut = EPI == kEpiSwiglu ? CW / 2 : CW;          // output columns per item
  constexpr int kRPL = CW == 64 ? 8 : 4;                         // NN: k-rows per 1 KB line
  static_assert(CW != 256 || (LAY == kLayNN && EPI == kEpiSwiglu), "256 columns: gate and up halves");
  const int G = gridDim.x;
  const int n_ct = (p.N + kOut - 1) / kOut;
  const int total = id1 - id0;
  // 128 columns: neighbouring items on different dies, as the dispatcher deals them; 64 columns: on one die, whose L2 then
  // serves both halves of a line that two items share
  auto tile_of = [&](int it) __attribute__((always_inline)) {
    const int id = it * G + b;
    return CW != 64 ? (id < total ? id : -1) : xcd_spread_tile(it, b, G, total);
  };
  int n_items = (total + G - 1) / G;
  if (n_items > 0 && tile_of(n_items - 1) < 0) --n_items;
  if (n_items <= 0) return;
  const int n_steps = (p.K + S::kKB - 1) / S::kKB;
  const int n_total = __builtin_amdgcn_readfirstlane(n_items * n_steps);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const lds_i32_ptr s_expert = (lds_i32_ptr)(smem + kStreamTables), s_row0 = s_expert + kMaxE, s_rows = s_row0 + kMaxE;
  const lds_i32_ptr s_tok = (lds_i32_ptr)(smem + kStreamGatherOff);
  const uint32_t lds0 = lds_addr_of(smem);
  const int ldb_bytes = p.ldb * 2;

  // ---- request side: item and step of the next stage to request ----
  const int r8 = lane >> 3;                                      // row of this lane inside an 8-row line
  struct { const char *a_base, *b_base; uint32_t a_off[AL], b_off[LAY == kLayNT ? 4 : S::kNB]; int step, item, slot; } q;
  q.step = 0; q.item = 0; q.slot = 0;
  auto item_of = [&](int it, int& ae, int& ct) __attribute__((always_inline)) {
    const int id = id0 + tile_of(it);
    ae = __builtin_amdgcn_readfirstlane(id / n_ct);
    ct = __builtin_amdgcn_readfirstlane(id - ae * n_ct);
  };
  auto set_item = [&]() __attribute__((always_inline)) {
    int ae, ct;
    item_of(q.item, ae, ct);
    const int e = __builtin_amdgcn_readfirstlane(s_expert[ae]), row0 = __builtin_amdgcn_readfirstlane(s_row0[ae]);
    const int rows = __builtin_amdgcn_readfirstlane(s_rows[ae]);
    const bool gathered = LAY == kLayNN && p.gather != nullptr;
    q.a_base = uniform_ptr(reinterpret_cast<const char*>(gathered ? p.A : p.A + (size_t)row0 * p.lda));
    q.b_base = uniform_ptr(reinterpret_cast<const char*>(p.B + (size_t)e * p.strideB));
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      // activation line wave + 4 i: CW = 128: rows 8 (wave + 4 i) ..; CW = 64: rows 8 ((wave + 4 i) / 2) .., k half wave & 1
      const int rl = CW != 64 ? wave + 4 * i : (wave + 4 * i) >> 1;
      const int row = min(rl * 8 + r8, rows - 1);                // rows past the end repeat the last one; never stored
      int arow = row;
      if (gathered) arow = row0 + row < kStreamGather ? s_tok[row0 + row] : p.gather[row0 + row];
      const int chunk = (lane & 7) ^ ((4 * (rl & 1) + (r8 >> 1)) & 7);
      q.a_off[i] = (uint32_t)(((long)arow * p.lda + chunk * 8) * 2);
    }
    if constexpr (LAY == kLayNN) {
      int kk, col;
      if (CW == 256) {
        // two lines per four k-rows: 128 gate columns, 128 up columns (chunks in the order that keeps the reads apart)
        kk = lane >> 4;
        const int c = ((lane & 15) - 4 * kk) & 15;
        col = min(ct * 128 + c * 8, p.N - 8);
        q.b_off[S::kNB - 1] = (uint32_t)((kk * p.ldb + p.N + min(ct * 128 + (c ^ 2) * 8, p.N - 8)) * 2);
      } else if (CW == 128) {
        kk = lane >> 4;
        const int c = ((lane & 15) - 4 * kk) & 15;               // staged chunk of 8 columns, k-rows rotated by 64 bytes
        if (EPI == kEpiSwiglu) col = c < 8 ? ct * 64 + c * 8 : p.N + ct * 64 + ((c - 8) ^ 2) * 8;
        else col = min(ct * 128 + c * 8, p.N - 8);
      } else {
        kk = r8;
        const int c = (lane & 7) ^ (4 * ((kk >> 1) & 1));
        if (EPI == kEpiSwiglu) col = c < 4 ? ct * 32 + c * 8 : p.N + ct * 32 + ((c - 4) ^ 2) * 8;
        else col = ct * 64 + c * 8;
      }
      q.b_off[0] = (uint32_t)((kk * p.ldb + col) * 2);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // weight line wave * 4 + i: 8 output columns x 64 k; CW = 64: column group (line / 2), k half line & 1
        const int nl = CW == 128 ? wave * 4 + i : wave * 2 + (i >> 1);
        const int n = min(ct * CW + nl * 8 + r8, p.N - 1);
        const int chunk = (lane & 7) ^ ((4 * (nl & 1) + (r8 >> 1)) & 7);
        q.b_off[i] = (uint32_t)(((size_t)n * p.ldb + chunk * 8) * 2);
      }
    }
  };
  auto request = [&](bool rows = true, bool weights = true) __attribute__((always_inline)) {   // both constant in a call
    if (q.step == 0) set_item();
    const int k0 = q.step * S::kKB;
    const uint32_t st = uniform_u32(lds0 + (uint32_t)(q.slot * S::kStage));
    // k past the end (an odd number of 64s with 128 to a stage): the last 64 again, not multiplied
    const char* a_k = uniform_ptr(q.a_base + (size_t)(CW != 64 ? k0 : min(k0 + (wave & 1) * 64, p.K - 64)) * 2);
#pragma unroll
    for (int i = 0; i < AL; ++i)
      if (rows) lds_dma16(a_k, q.a_off[i], st + (S::kALine0 + wave + 4 * i) * kLine);
#pragma unroll
    for (int i = 0; i < S::kBLoads; ++i) {
      const char* b_k;
      if (CW == 256) b_k = q.b_base + (size_t)(k0 + (wave * 4 + (i >> 1)) * 4) * ldb_bytes;
      else if (LAY == kLayNN) b_k = q.b_base + (size_t)min(k0 + (wave * 4 + i) * kRPL, p.K - kRPL) * ldb_bytes;
      else b_k = q.b_base + (size_t)(CW == 128 ? k0 : min(k0 + (i & 1) * 64, p.K - 64)) * 2;
      if (weights) lds_dma16<CW != 64>(uniform_ptr(b_k), q.b_off[LAY == kLayNT ? i : CW == 256 ? i & 1 : 0], st + (wave * S::kBLoads + i) * kLine);
    }
    q.slot = q.slot == S::kDepth - 1 ? 0 : q.slot + 1;
    if (++q.step == n_steps) { q.step = 0; ++q.item; }
  };

  // ---- operand reads: offsets of this lane inside a stage ----
  const int blk = CW != 64 ? wave : wave & 1;                    // this wave's (first) 32-column block; the second: blk + 4
  const bool active = CW != 64 || S::kWaveRows == 2 || wave < 2;
  const int mt0 = S::kWaveRows == 2 ? (wave >> 1) * S::kMTW : 0;  // this wave's first row block
  uint32_t b_rd;
  if (LAY == kLayNN) {
    const int g = lane >> 4, i = lane & 15, kk = i >> 2;
    int c;                                                       // staged chunk of this 16-lane group's columns
    if (CW == 256) c = (2 * blk + ((i & 3) >> 1)) ^ ((g & 1) * 2);   // gate line, up line
    else if (EPI == kEpiSwiglu) c = (g & 1) ? CW / 16 + ((2 * blk + ((i & 3) >> 1)) ^ 2) : 2 * blk + ((i & 3) >> 1);
    else c = 4 * blk + (g & 1) * 2 + ((i & 3) >> 1);
    if (CW == 256) b_rd = (uint32_t)(((g >> 1) * 4 + (g & 1)) * kLine + kk * 256 + ((c + 4 * kk) & 15) * 16 + (i & 1) * 8);
    else if (CW == 128) b_rd = (uint32_t)((g >> 1) * 2 * kLine + kk * 256 + ((c + 4 * kk) & 15) * 16 + (i & 1) * 8);
    else b_rd = (uint32_t)((g >> 1) * kLine + kk * 128 + (c ^ (4 * ((kk >> 1) & 1))) * 16 + (i & 1) * 8);
  } else {
    b_rd = (uint32_t)((blk * 4 + (l32 >> 3)) * (CW != 64 ? 1 : 2) * kLine + (l32 & 7) * 128);
  }
  const int ar = l32 & (S::kRows < 32 ? S::kRows - 1 : 31);      // 16-row stages: the upper lanes repeat the rows
  constexpr int kABlock = (CW != 64 ? 4 : 8) * kLine;            // activation lines of 32 rows
  const uint32_t a_rd = (uint32_t)(S::kALine0 * kLine + mt0 * kABlock + (ar >> 3) * (CW != 64 ? 1 : 2) * kLine + (ar & 7) * 128);
  const int a_sw = (ar >> 1) & 7, b_sw = (l32 >> 1) & 7;

  f32x16 acc[S::kNB][S::kMTW];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < S::kNB; ++nb)
#pragma unroll
      for (int mt = 0; mt < S::kMTW; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][mt][r] = 0.f;
  };
  clear();

  auto half_stage = [&](lds_cptr st, int h) __attribute__((always_inline)) {   // 64 k: four MFMA slices
    bf16x8 wf[S::kNB][4], xf[4][S::kMTW];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int ks = h * 4 + s;
      if (LAY == kLayNN) {
#pragma unroll
        for (int nb = 0; nb < S::kNB; ++nb) {
          // the second block's 64 columns further on are 8 chunks on, and a line's 16 chunks wrap around
          const lds_cptr b = st + (nb ? b_rd ^ 128u : b_rd) + ks * (CW == 256 ? 8 : CW == 128 ? 4 : 2) * kLine;
          wf[nb][s] = join_tr(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)b),
                              __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(b + (CW == 256 ? 2 * kLine : CW == 128 ? kLine : kLine / 2))));
        }
      } else {
        wf[0][s] = *(lds_bf16x8_cptr)(st + b_rd + h * kLine + (uint32_t)(((s * 2 + lh) ^ b_sw) << 4));
      }
#pragma unroll
      for (int mt = 0; mt < S::kMTW; ++mt)
        xf[s][mt] = *(lds_bf16x8_cptr)(st + a_rd + h * kLine + mt * kABlock + (uint32_t)(((s * 2 + lh) ^ a_sw) << 4));
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int mt = 0; mt < S::kMTW; ++mt)
#pragma unroll
        for (int nb = 0; nb < S::kNB; ++nb) acc[nb][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[nb][s], xf[s][mt], acc[nb][mt], 0, 0, 0);
  };

  if constexpr (ROLE == kStreamSecond) {
    const auto q0 = q;
    for (int g = 0; g < S::kDepth - 1 && g < n_total; ++g) request(false, true);
    if (!ready()) {
      wait_vmcnt<0>();
      return;
    }
    q = q0;
    for (int g = 0; g < S::kDepth - 1 && g < n_total; ++g) request(true, false);
    wait_vmcnt<0>();                                             // the waits below count whole stages in order
  } else {
    for (int g = 0; g < S::kDepth - 1 && g < n_total; ++g) request();
  }
  int step = 0, item = 0, slot = 0;
  for (int g = 0; g < n_total; ++g) {
    stream_wait<S::kLoads, S::kDepth - 2>(n_total - 1 - g);      // this wave's part of stage g has landed
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();                                // ... and everybody's; stage g - 1 has been read by all
    if (g + S::kDepth - 1 < n_total) request();                  // into the slot of stage g - 1
    if (active) {
      const lds_cptr st = (lds_cptr)smem + slot * S::kStage;
      half_stage(st, 0);
      if (CW == 64 && step * S::kKB + 64 < p.K) half_stage(st, 1);
    }
    slot = slot == S::kDepth - 1 ? 0 : slot + 1;
    if (++step < n_steps) continue;
    step = 0;
    int ae, ct;
    item_of(item++, ae, ct);
    if (!active) continue;
    const int row0 = __builtin_amdgcn_readfirstlane(s_row0[ae]), rows = __builtin_amdgcn_readfirstlane(s_rows[ae]);
    // lane: row l32 of each 32-row block; register group q: staged columns q * 8 + lh * 4 .. + 3 of the wave's block
#pragma unroll
    for (int mt = 0; mt < S::kMTW; ++mt) {
      const int m = (mt0 + mt) * 32 + l32;
      const size_t grow = (size_t)(row0 + m);
      if (m < rows) {
        if (EPI == kEpiSwiglu) {
#pragma unroll
          for (int qb = 0; qb < 2 * S::kNB; ++qb) {
            const int nb = qb >> 1, qg = qb & 1;
            const int c = ct * kOut + (blk + 4 * nb) * 16 + qg * 8 + lh * 4;
            if (CW == 256 && c >= p.N) continue;
            float gt[4], u[4], a[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              gt[x] = acc[nb][mt][qg * 4 + x];
              u[x] = acc[nb][mt][qg * 4 + 8 + x];
              a[x] = gt[x] * sigmoid_bf16_(gt[x]) * u[x];
            }
            store8<ROLE != kStreamAlone>(p.C + grow * p.ldc + c, u32x2{pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3])});
            if (p.C2) {
              __bf16* h = p.C2 + grow * (size_t)(2 * p.N) + c;
              *reinterpret_cast<u32x2*>(h) = u32x2{pack_bf16(gt[0], gt[1]), pack_bf16(gt[2], gt[3])};
              *reinterpret_cast<u32x2*>(h + p.N) = u32x2{pack_bf16(u[0], u[1]), pack_bf16(u[2], u[3])};
            }
          }
        } else {
#pragma unroll
          for (int qg = 0; qg < 4; ++qg) {
            const int c = ct * kOut + blk * 32 + qg * 8 + lh * 4;
            if (c >= p.N) continue;
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) v[x] = acc[0][mt][qg * 4 + x];
            if (EPI == kEpiSwigluGrad) {
              const __bf16* h = p.G + grow * (size_t)(2 * p.N) + c;
              float dg[4], du[4];
              swiglu_grad4(v, *reinterpret_cast<const u32x2*>(h), *reinterpret_cast<const u32x2*>(h + p.N), dg, du);
              __bf16* o = p.C + grow * p.ldc + c;
              *reinterpret_cast<u32x2*>(o) = u32x2{pack_bf16(dg[0], dg[1]), pack_bf16(dg[2], dg[3])};
              *reinterpret_cast<u32x2*>(o + p.N) = u32x2{pack_bf16(du[0], du[1]), pack_bf16(du[2], du[3])};
            } else {
              store8<ROLE != kStreamAlone>(p.C + grow * p.ldc + c, u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])});
            }
          }
        }
      }
    }
    clear();
  }
}

// The same with stages of ROWS activation rows.
template <int LAY, int EPI, int CW, int ROWS, int ROLE, typename Ready>
__device__ __forceinline__ void stream_rows(const GemmParams& p, int id0, int id1, int b, char* smem, Ready&& ready) {
  constexpr int AL = ROWS / (CW == 64 ? 16 : 32);
  static_assert(StreamShape<CW, AL>::kRows == ROWS, "rows of a stage");
  stream_items<LAY, EPI, CW, AL, ROLE>(p, id0, id1, b, smem, ready);
}

// Whole launch of a grouped GEMM that stream_takes, in the form of stream_form.  The comparisons of max_rows below are those of
// stream_stage_rows.
static_assert(stream_stage_rows(64, 16) == 16 && stream_stage_rows(64, 17) == 32 && stream_stage_rows(64, 32) == 32 &&
              stream_stage_rows(64, 33) == 64 && stream_stage_rows(64, 64) == 64 && stream_stage_rows(64, 65) == 128, "64 columns");
static_assert(stream_stage_rows(128, 32) == 32 && stream_stage_rows(128, 33) == 64 && stream_stage_rows(128, 64) == 64 &&
              stream_stage_rows(128, 65) == 128 && stream_stage_rows(256, 32) == 32 && stream_stage_rows(256, 33) == 64, "128, 256");
// Tables in LDS: experts with rows, in expert order (every wave counts, wave 0 writes), and the tokens of the first rows if the
// activations are gathered.  Returns the number of such experts.
__device__ __forceinline__ int stream_tables(const int32_t* offsets, int E_local, const int32_t* gather, char* smem) {
  const int lane = lane_id();
  const lds_i32_ptr s_expert = (lds_i32_ptr)(smem + kStreamTables), s_row0 = s_expert + kMaxE, s_rows = s_row0 + kMaxE;
  int n_act = 0, R = 0;
  auto fill = [&](auto passes) __attribute__((always_inline)) {   // 64 experts each
    constexpr int P = decltype(passes)::value;
    int lo[P], hi[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int e = i * kWave + lane;
      lo[i] = e < E_local ? offsets[e] : 0;
      hi[i] = e < E_local ? offsets[e + 1] : 0;
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const uint64_t bal = __ballot(hi[i] > lo[i]);
      const int at = n_act + __popcll(bal & ((1ull << lane) - 1));
      if (threadIdx.x < kWave && hi[i] > lo[i]) {
        s_expert[at] = i * kWave + lane;
        s_row0[at] = lo[i];
        s_rows[at] = hi[i] - lo[i];
      }
      n_act += __popcll(bal);
    }
  };
  if (E_local <= kWave) fill(std::integral_constant<int, 1>{});
  else fill(std::integral_constant<int, kMaxE / kWave>{});
  if (gather) {
    R = offsets[E_local];
    const lds_i32_ptr s_tok = (lds_i32_ptr)(smem + kStreamGatherOff);
    for (int i = threadIdx.x; i < min(R, kStreamGather); i += kGemmThreads) s_tok[i] = gather[i];
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(n_act);
}

// The share of workgroup b, in the form of stream_form (the roles of the single launch: up to 64 rows).
template <int LAY, int EPI, int ROLE, typename Ready>
__device__ __forceinline__ void stream_share(const GemmParams& p, int max_rows, int n_act, int b, char* smem, Ready&& ready) {
  const int G = gridDim.x;
  const bool narrow = stream_narrow(n_act, p.N, EPI == kEpiSwiglu, G);
  if constexpr (LAY == kLayNN && EPI == kEpiSwiglu) {
    const int n256 = n_act * stream_tiles(p.N, 128), n128 = n_act * stream_tiles(p.N, 64);
    if (!narrow && stream_wide(max_rows, n256, n128, p.N, G)) {
      const int whole = stream_whole(n256, n128, G);
      if (max_rows > 32) stream_rows<LAY, EPI, 256, 64, ROLE>(p, 0, whole, b, smem, ready);
      else stream_rows<LAY, EPI, 256, 32, ROLE>(p, 0, whole, b, smem, ready);
      if (whole == n256) return;
      __syncthreads();                                           // the ring has been read out by all
      if (max_rows > 32) stream_rows<LAY, EPI, 128, 64, ROLE>(p, 2 * whole, 2 * n256, b, smem, ready);
      else stream_rows<LAY, EPI, 128, 32, ROLE>(p, 2 * whole, 2 * n256, b, smem, ready);
      return;
    }
  }
  constexpr int kOut64 = EPI == kEpiSwiglu ? 32 : 64;
  const int total = n_act * stream_tiles(p.N, narrow ? kOut64 : 2 * kOut64);
  if (narrow) {
    if (ROLE == kStreamAlone && max_rows > 64) stream_rows<LAY, EPI, 64, 128, ROLE>(p, 0, total, b, smem, ready);
    else if (max_rows > 32) stream_rows<LAY, EPI, 64, 64, ROLE>(p, 0, total, b, smem, ready);
    else if (max_rows > 16) stream_rows<LAY, EPI, 64, 32, ROLE>(p, 0, total, b, smem, ready);
    else stream_rows<LAY, EPI, 64, 16, ROLE>(p, 0, total, b, smem, ready);
  } else {
    if (ROLE == kStreamAlone && max_rows > 64) stream_rows<LAY, EPI, 128, 128, ROLE>(p, 0, total, b, smem, ready);
    else if (max_rows > 32) stream_rows<LAY, EPI, 128, 64, ROLE>(p, 0, total, b, smem, ready);
    else stream_rows<LAY, EPI, 128, 32, ROLE>(p, 0, total, b, smem, ready);
  }
}

template <int LAY, int EPI>
__device__ __forceinline__ void stream_gemm_bf16(const GemmParams& p, int max_rows, char* smem) {
  const int n_act = stream_tables(p.offsets, p.E_local, LAY == kLayNN ? p.gather : nullptr, smem);
  stream_share<LAY, EPI, kStreamAlone>(p, max_rows, n_act, blockIdx.x, smem, [] { return true; });
}

}  // namespace moe
