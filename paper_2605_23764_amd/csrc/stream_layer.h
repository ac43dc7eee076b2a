// Dispatch to Combine of up to 64 tokens as ONE launch (MOE_MODE_PERSISTENT, bf16): no expert has more than 64 rows, so both GEMMs run
// as weight streams (gemm_stream.h) instead of tile tasks.
//
// Every workgroup runs a share of GEMM-1's items, then one of GEMM-2's, then combines a few tokens.  In front of GEMM-2 and of
// Combine the whole launch meets: a workgroup counts its share done once the results, stored through to memory, have been
// acknowledged, and who needs them polls the eight counts (one per class of workgroups, id % 8).  GEMM-2's weights do not depend on
// that: a workgroup has as many of them under way as its ring holds when it starts to wait.
// Shares are drawn from counters, not fixed by the workgroup's id: a workgroup draws one of either GEMM when it starts, and before it
// waits it runs those that nobody has drawn.  So whoever waits waits for workgroups that are running and do not wait for it,
// however few of them fit on the chip beside other work.
// What bounds it: the weight streams, and two meetings of 3..5 us: stores acknowledged, count, poll, first activations.
// Measured, layer, same bits, against tile tasks: H = 2048, I = 1408, 16 experts, k = 4: T = 1 75.5 -> 36.9 us, T = 8 91 -> 65, T = 64
// 100 -> 79; H = 7168, I = 2048, 32 of 256 experts, k = 8: T = 4 159 -> 100, T = 32 391 -> 337, T = 64 540 -> 436.  The four launches of
// the serialized mode take 35, 56, 61 and 328 and 426 us (T = 1, 8, 64; 32, 64): a launch's end and start cost less than a
// meeting, so that mode keeps them.  As a branch of the tile kernel, for any T with up to 64 rows per expert, its loops had
// spilled registers: T = 1 45 us, T = 1000 587 -> 637.
#pragma once
#include "gemm_stream.h"
#include "permute_combine.h"
#include "persistent.h"
#include "wave_sync.h"

namespace moe {

// Counters, zero at the start: where the tile tasks have their events; eight words each, on lines of their own.
constexpr int kEvStreamDraw = kEvPerTile, kEvStreamDone1 = kEvPerTile + 32, kEvStreamDone2 = kEvPerTile + 64;
constexpr int kStreamLayerEvents = kEvStreamDone2 + kNumXcd;
static_assert(kStreamLayerEvents <= kEvPerTile + 2 * (2 + kMapSlack), "the events of the smallest layer");

struct StreamLayerParams {
  GemmParams g1, g2;       // g1 gathers its rows from the tokens
  PermuteParams perm;      // copy: the permuted tokens are an output as well
  CombineParams comb;
  uint32_t* events;
  int32_t* meta;
  int copy;
  uint32_t spin_limit;
  int32_t timeout_status;
};

__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void stream_layer_kernel(StreamLayerParams sp) {
  __shared__ __attribute__((aligned(1024))) char smem[kGemmLdsBytes];
  volatile int* s_box = reinterpret_cast<volatile int*>(smem + kStreamBox);
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int G = gridDim.x, W = G / kNumXcd, b = blockIdx.x, q = b % kNumXcd;
  const int max_rows = __builtin_amdgcn_readfirstlane(sp.meta[kMetaMaxRows]);
  // words 0..7: shares of GEMM-1 drawn, 8..15: of GEMM-2, 16..23: workgroups started
  uint32_t* const draw = sp.events + kEvStreamDraw;
  uint32_t mine = 0;
  if (wave == 0 && lane < 3) mine = __hip_atomic_fetch_add(draw + 8 * lane + q, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int n_act = stream_tables(sp.g1.offsets, sp.g1.E_local, sp.g1.gather, smem);
  if (wave == 0) {
    s_box[0] = __builtin_amdgcn_readlane((int)mine, 0);
    s_box[1] = __builtin_amdgcn_readlane((int)mine, 1);
    s_box[2] = __builtin_amdgcn_readlane((int)mine, 2);
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(s_box[2]) >= W) return;       // a second launch on the same routing: nothing is left to do
  const int first1 = __builtin_amdgcn_readfirstlane(s_box[0]), first2 = __builtin_amdgcn_readfirstlane(s_box[1]);
  // Every wave has read the box before wave 0 writes it again: with a drawn share of GEMM-1 that is somebody else's by now (>= W, as for
  // a workgroup that starts late) there is no work, and with it no barrier, in front of that.  Every later read has one behind it.
  __syncthreads();
  if (sp.copy) {
    const int R = sp.meta[kMetaRows], nw = blockDim.x / kWave;
    for (int r0 = b * nw; r0 < R; r0 += G * nw) permute_rows<4>(sp.perm, r0, min(R, r0 + nw), wave, nw);
  }
  // lane i < 8: counter i; the others: full
  auto counts = [&](const uint32_t* c) __attribute__((always_inline)) {
    return lane < kNumXcd ? __hip_atomic_load(c + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (uint32_t)W;
  };
  // The share drawn at the start, then what nobody has drawn.  done: one count per share.  work: false, it has given up (all waves
  // alike); its share stays uncounted, so that every wait for the results expires as well and nobody goes on with rows that were
  // never stored (out is left as it was), and the workgroup is done.
  auto shares = [&](uint32_t* dr, int first, uint32_t* done, auto&& work) __attribute__((always_inline)) {
    int t = first, c = q;
    for (;;) {
      if (t < W) {
        if (!work(t * kNumXcd + c)) return false;
        wait_own_stores();
        __syncthreads();                   // ... every wave's, and the ring has been read out
      }
      if (wave == 0) {
        if (t < W && lane == 0) __hip_atomic_fetch_add(done + c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t left = __ballot(counts(dr) < (uint32_t)W);
        int cls = -1, tk = W;
        if (left) {                        // never as long as the whole grid fits on the chip
          cls = (int)__builtin_ctzll(left);
          tk = (int)wave_atomic_add(dr + cls, 1u);
        }
        s_box[0] = tk;
        s_box[1] = cls;
      }
      __syncthreads();
      t = __builtin_amdgcn_readfirstlane(s_box[0]);
      c = __builtin_amdgcn_readfirstlane(s_box[1]);
      __syncthreads();
      if (c < 0) return true;
    }
  };
  auto wait_all = [&](const uint32_t* done) __attribute__((always_inline)) {   // bounded; false: given up, status set
    if (wave == 0) {
      uint32_t polls = 0;
      int ok = 1;
      while (__ballot(counts(done) < (uint32_t)W)) {
        if (++polls > sp.spin_limit) { ok = 0; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      if (!ok) __hip_atomic_store(&sp.meta[kMetaStatus], sp.timeout_status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_box[0] = ok;
    }
    __syncthreads();
    const int ok = __builtin_amdgcn_readfirstlane(s_box[0]);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // lines of the result that this die has written a part of
    __syncthreads();
    return ok;
  };
  shares(draw, first1, sp.events + kEvStreamDone1, [&](int v) __attribute__((always_inline)) {
    stream_share<kLayNN, kEpiSwiglu, kStreamFirst>(sp.g1, max_rows, n_act, v, smem, [] { return true; });
    return true;
  });
  int a_ready = -1;                        // -1: not asked yet
  const bool stored = shares(draw + 8, first2, sp.events + kEvStreamDone2, [&](int v) __attribute__((always_inline)) {
    stream_share<kLayNN, kEpiStore, kStreamSecond>(sp.g2, max_rows, n_act, v, smem, [&]() __attribute__((always_inline)) {
      if (a_ready < 0) a_ready = wait_all(sp.events + kEvStreamDone1);
      return a_ready != 0;
    });
    return a_ready != 0;
  });
  if (!stored || b >= sp.comb.T || !wait_all(sp.events + kEvStreamDone2)) return;
  for (int t = b + wave * G; t < sp.comb.T; t += G * (int)(blockDim.x / kWave)) {
    int rowv;
    float wv;
    combine_load_slots(sp.comb, t, rowv, wv);
    with_row_vectors(sp.comb.H / 8, [&](auto uv) { combine_token_rows<true, decltype(uv)::value, 4>(sp.comb, t, rowv, wv); });
  }
}

}  // namespace moe
