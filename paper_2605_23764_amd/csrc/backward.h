// Backward-only operators (paper Section 2.2, Figure 2b): backward Dispatch (the
// gradient of the forward Combine) and the fp32 versions of the four backward
// GEMMs.  The bf16 GEMMs are the NT / TN layouts of gemm_bf16.h; backward Combine
// (the gradient of the forward Dispatch) is combine_token with unit weights.
#pragma once
#include "common.h"
#include "gemm_f32.h"
#include "route.h"

namespace moe {

struct BwdDispatchParams {
  const void* dY;          // [T,H]
  const void* Yp;          // [R_max,H] saved GEMM-2 output
  void* dYp;               // [R_max,H]
  const int32_t* row_of;   // [T,k]
  const float* topk_w;     // [T,k]
  float* d_topk_w;         // [T,k]
  int T, H, k;
  // The backward's M-tile map, rebuilt from the saved rows per expert, and the counters the later kernels draw
  // tickets from: nothing in this kernel needs them, so its first workgroup makes them on the side (one wave).
  const int32_t* counts;   // [E_local]
  int E_local, wide_max, granule, tall;
  TileMap tiles;
  uint32_t* zero;
  int n_zero;
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// One wave per token t: for every local slot j with row r = row_of[t,j]
//   dYp[r,:] = topk_w[t,j] * dY[t,:],   d_topk_w[t,j] = <dY[t,:], Yp[r,:]>  (fp32),
// and d_topk_w[t,j] = 0 for slots whose expert is not local.
// Lane j < k holds slot j; the local slots are walked through the ballot of "row >= 0" with rows and
// weights as wave-uniform scalars.  A pass covers 7 x 64 16-byte vectors of the row: dY[t] is fetched
// once per pass and reused by every local slot, the Yp vectors of a slot are all in flight together.
template <bool BF16>
__device__ __forceinline__ void bwd_dispatch_token(const BwdDispatchParams& p, int t) {
  const int lane = lane_id();
  int rowv = -1;
  float wv = 0.f;
  if (lane < p.k) {
    rowv = p.row_of[(size_t)t * p.k + lane];
    wv = p.topk_w[(size_t)t * p.k + lane];
    if (rowv < 0) p.d_topk_w[(size_t)t * p.k + lane] = 0.f;
  }
  const uint64_t local = __ballot(rowv >= 0);
  if (local == 0) return;
  constexpr int EPV = BF16 ? 8 : 4;                 // elements per 16-byte vector
  constexpr int U = BF16 ? 7 : 4;                   // vectors per lane per pass
  const int vec = p.H / EPV;
  const size_t row_bytes = (size_t)p.H * (BF16 ? 2 : 4);
  const uint4* dy = reinterpret_cast<const uint4*>(static_cast<const char*>(p.dY) + (size_t)t * row_bytes);
  float dot[kMaxK];
#pragma unroll
  for (int n = 0; n < kMaxK; ++n) dot[n] = 0.f;
  for (int v0 = lane; v0 < vec; v0 += U * kWave) {
    uint4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = v0 + u * kWave < vec ? dy[v0 + u * kWave] : make_uint4(0, 0, 0, 0);
    uint64_t m = local;
#pragma unroll
    for (int n = 0; n < kMaxK; ++n) {
      if (m == 0) break;
      const int j = __builtin_amdgcn_readfirstlane(__builtin_ctzll(m));
      m &= m - 1;
      const int r = __builtin_amdgcn_readlane(rowv, j);
      const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wv), j));
      const uint4* yp = reinterpret_cast<const uint4*>(static_cast<const char*>(p.Yp) + (size_t)r * row_bytes);
      uint4* o = reinterpret_cast<uint4*>(static_cast<char*>(p.dYp) + (size_t)r * row_bytes);
      uint4 b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = v0 + u * kWave < vec ? yp[v0 + u * kWave] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (v0 + u * kWave >= vec) break;
        const uint32_t aw[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
        const uint32_t bw[4] = {b[u].x, b[u].y, b[u].z, b[u].w};
        uint32_t ow[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          if constexpr (BF16) {
            const float lo = bf16_lo(aw[x]), hi = bf16_hi(aw[x]);
            dot[n] = fmaf(lo, bf16_lo(bw[x]), dot[n]);
            dot[n] = fmaf(hi, bf16_hi(bw[x]), dot[n]);
            ow[x] = pack_bf16(w * lo, w * hi);
          } else {
            const float av = __builtin_bit_cast(float, aw[x]);
            dot[n] = fmaf(av, __builtin_bit_cast(float, bw[x]), dot[n]);
            ow[x] = __builtin_bit_cast(uint32_t, w * av);
          }
        }
        o[v0 + u * kWave] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
      }
    }
  }
  uint64_t m = local;
#pragma unroll
  for (int n = 0; n < kMaxK; ++n) {
    if (m == 0) break;
    const int j = __builtin_amdgcn_readfirstlane(__builtin_ctzll(m));
    m &= m - 1;
    const float d = wave_sum(dot[n]);
    if (lane == 0) p.d_topk_w[(size_t)t * p.k + j] = d;
  }
}

// Workgroup 0 makes the map and the counters (true); it is the first to start, so its serial chain runs under the rows of the others.
template <bool BF16>
__device__ __forceinline__ bool bwd_dispatch(const BwdDispatchParams& p) {
  const int n_waves = blockDim.x / kWave;
  const int wave = threadIdx.x / kWave;
  if (blockIdx.x == 0) {
    if (wave == 0) {
      for (int i = threadIdx.x; i < p.n_zero; i += kWave) p.zero[i] = 0;
      build_tile_map(p.E_local, p.counts, p.wide_max, p.granule, p.tall, nullptr, nullptr, p.tiles);
    }
    return true;
  }
  const int n_blocks = (int)gridDim.x - 1;
  for (int t = ((int)blockIdx.x - 1) * n_waves + wave; t < p.T; t += n_blocks * n_waves) bwd_dispatch_token<BF16>(p, t);
  return false;
}

template <bool BF16>
__global__ __launch_bounds__(256) void bwd_dispatch_kernel(BwdDispatchParams p) { bwd_dispatch<BF16>(p); }

// ---- fp32 backward GEMMs on the tile of gemm_f32.h (H and I are multiples of 64: every tile is full in N, and in M
// except for the last rows of an expert's segment) ----
struct GemmBwdParamsF32 {
  const float* A;     // dgrad: [rows, lda]; wgrad: [rows, lda] read transposed
  const float* B;     // dgrad: per expert [N, ldb] (weights, read transposed); wgrad: [rows, ldb]
  float* C;           // dgrad: [rows, ldc]; wgrad: per expert [M, ldc]
  const float* G;     // SwiGLU-grad: saved pre-activations [rows, 2N]
  long strideB, strideC;
  int K, N, M;
  int lda, ldb, ldc;
  int n_ntiles, n_mtiles, E_local;
  const int32_t* offsets;
  TileMap tiles;
};

// One result v of a data gradient (SwiGLU-grad: v = dA).
template <int EPI>
__device__ __forceinline__ void store_dgrad_f32(const GemmBwdParamsF32& p, size_t grow, int c, float v) {
  if (EPI == kEpiSwigluGrad) {
    const float g = p.G[grow * (size_t)(2 * p.N) + c], u = p.G[grow * (size_t)(2 * p.N) + p.N + c];
    const float s = sigmoidf_(g);
    p.C[grow * p.ldc + c] = v * u * s * (1.f + g * (1.f - s));
    p.C[grow * p.ldc + p.N + c] = v * g * s;
  } else {
    p.C[grow * p.ldc + c] = v;
  }
}

// act_grad (+ SwiGLU_grad) and gate_grad: C[rows, N] = A[rows, K] * W_e[N, K]^T per M tile.
template <int EPI>
__device__ __forceinline__ void dgrad_f32(const GemmBwdParamsF32& p, int b, float* smem) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  auto whole = [&](int tile) __attribute__((always_inline)) {
    const int mtile = tile / p.n_ntiles, n0 = (tile % p.n_ntiles) * kFBN;
    const int e = p.tiles.expert[mtile], row0 = p.tiles.row0[mtile], rows = p.tiles.rows[mtile];
    if (rows <= 0) return;   // the empty half of a pair slot (block-uniform)
    f32x16 acc[1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = 0.f;
    gemm_rows_f32<true, true, 1>(acc, p.A + (size_t)(row0 + min(tid >> 2, rows - 1)) * p.lda + (tid & 3) * 4, 1,
                                 p.B + (size_t)e * p.strideB + (size_t)(n0 + (tid >> 2)) * p.ldb + (tid & 3) * 4, 1, 0, p.K,
                                 wm * 32 < rows, smem);
    const int c = n0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = wm * 32 + f32_acc_row(r, lane);
      if (m < rows) store_dgrad_f32<EPI>(p, (size_t)(row0 + m), c, acc[0][r]);
    }
  };
  auto quarter = [&](int tile, int qm, int qn) __attribute__((always_inline)) {
    const int mtile = tile / p.n_ntiles, n0 = (tile % p.n_ntiles) * kFBN + qn * 32;
    const int e = p.tiles.expert[mtile], row0 = p.tiles.row0[mtile] + qm * 32, rows = p.tiles.rows[mtile] - qm * 32;
    if (rows <= 0) return;
    f32x4 acc[1] = {{0.f, 0.f, 0.f, 0.f}};
    gemm_core_f32_quarter<true, true, 1, false>(acc, p.A + (size_t)(row0 + min(tid >> 3, rows - 1)) * p.lda + (tid & 7) * 4, 1,
                                                p.B + (size_t)e * p.strideB + (size_t)(n0 + (tid >> 3)) * p.ldb + (tid & 7) * 4,
                                                1, 0, p.K, smem);
    const int c = n0 + wn * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = wm * 16 + 4 * (lane >> 4) + r;
      if (m < rows) store_dgrad_f32<EPI>(p, (size_t)(row0 + m), c, acc[0][r]);
    }
  };
  f32_sweeps(b, p.tiles.meta[kMetaMTiles] * p.n_ntiles, p.K, p.tiles.meta[kMetaMaxRows] <= 32, whole, quarter);
}

template <int EPI>
__global__ __launch_bounds__(256) void grouped_dgrad_f32_kernel(GemmBwdParamsF32 p) {
  __shared__ __attribute__((aligned(16))) float smem[kFLdsFloats1];
  dgrad_f32<EPI>(p, blockIdx.x, smem);
}

// w2_grad and w1_grad: C_e[M, N] = A_e[rows_e, M]^T * B_e[rows_e, N]; zeros for experts without rows.  A launch does one or
// both (NG), the second one's tiles behind the first one's: one partly filled last sweep instead of two (T = 256, H = 256,
// I = 128, 8 experts: training step 56.3 -> 52 us; T = 1500, H = 512, I = 448, 10 experts: backward 126 -> 116).
template <int NG>
struct WgradGroupF32 { GemmBwdParamsF32 p[NG]; };
template <int NG>
__device__ __forceinline__ void wgrad_f32(const WgradGroupF32<NG>& w, int b, float* smem) {
  const int per0 = w.p[0].n_mtiles * w.p[0].n_ntiles, total0 = w.p[0].E_local * per0;
  const int per1 = w.p[NG - 1].n_mtiles * w.p[NG - 1].n_ntiles, total1 = NG > 1 ? w.p[NG - 1].E_local * per1 : 0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  auto whole = [&](int t) __attribute__((always_inline)) {
    const int i = NG > 1 ? __builtin_amdgcn_readfirstlane(t >= total0 ? 1 : 0) : 0, tile = i ? t - total0 : t, per_e = i ? per1 : per0;
    const GemmBwdParamsF32& p = w.p[i];
    const int e = tile / per_e, rem = tile % per_e;
    const int m0 = (rem / p.n_ntiles) * kFBM, n0 = (rem % p.n_ntiles) * kFBN;
    const int seg0 = p.offsets[e], cnt = p.offsets[e + 1] - seg0;
    f32x16 acc[1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = 0.f;
    const size_t k0 = (size_t)(seg0 + (tid >> 4));
    gemm_core_f32<false, false, 1, true, true>(acc, p.A + k0 * p.lda + m0 + (tid & 15) * 4, p.lda,
                                               p.B + k0 * p.ldb + n0 + (tid & 15) * 4, p.ldb, 0, cnt, smem);
    float* c_base = p.C + (size_t)e * p.strideC + (size_t)(m0 + wm * 32) * p.ldc + n0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) c_base[(size_t)f32_acc_row(r, lane) * p.ldc] = acc[0][r];
  };
  auto quarter = [&](int t, int qm, int qn) __attribute__((always_inline)) {
    const int i = NG > 1 ? __builtin_amdgcn_readfirstlane(t >= total0 ? 1 : 0) : 0, tile = i ? t - total0 : t, per_e = i ? per1 : per0;
    const GemmBwdParamsF32& p = w.p[i];
    const int e = tile / per_e, rem = tile % per_e;
    const int m0 = (rem / p.n_ntiles) * kFBM + qm * 32, n0 = (rem % p.n_ntiles) * kFBN + qn * 32;
    const int seg0 = p.offsets[e], cnt = p.offsets[e + 1] - seg0;
    f32x4 acc[1] = {{0.f, 0.f, 0.f, 0.f}};
    const size_t k0 = (size_t)(seg0 + (tid >> 3));
    gemm_core_f32_quarter<false, false, 1, true>(acc, p.A + k0 * p.lda + m0 + (tid & 7) * 4, p.lda,
                                                 p.B + k0 * p.ldb + n0 + (tid & 7) * 4, p.ldb, 0, cnt, smem);
    float* c_base = p.C + (size_t)e * p.strideC + (size_t)(m0 + wm * 16 + 4 * (lane >> 4)) * p.ldc + n0 + wn * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) c_base[(size_t)r * p.ldc] = acc[0][r];
  };
  f32_sweeps(b, total0 + total1, w.p[0].offsets[w.p[0].E_local] / w.p[0].E_local, false, whole, quarter);
}

template <int NG>
__global__ __launch_bounds__(256) void grouped_wgrad_f32_kernel(WgradGroupF32<NG> w) {
  __shared__ __attribute__((aligned(16))) float smem[kFLdsFloats1];
  wgrad_f32<NG>(w, blockIdx.x, smem);
}

// gate_grad and both weight gradients, which only share inputs, as one launch behind dH1 (small layers, one stream): workgroups that gate_grad's
// last sweep leaves idle go on with the weight gradients.  Its sweeps are dealt in the other order inside a die, so that it is not
// the same workgroups that get one more tile of both.
__global__ __launch_bounds__(256) void grouped_grads_f32_kernel(GemmBwdParamsF32 gate, WgradGroupF32<2> w) {
  __shared__ __attribute__((aligned(16))) float smem[kFLdsFloats1];
  const int b = blockIdx.x;
  dgrad_f32<kEpiStore>(gate, ((int)(gridDim.x >> 3) - 1 - (b >> 3)) * 8 + (b & 7), smem);
  __syncthreads();                         // the stages have been read out
  wgrad_f32<2>(w, b, smem);
}

}  // namespace moe
