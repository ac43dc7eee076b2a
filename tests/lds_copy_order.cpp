// Runs the grouped bf16 GEMM kernel's own source on the CPU, one lane of each wave after the other, and checks the order of
// what it does to the LDS.  Arithmetic, memory and synchronisation are stubs; kept are the events of a wave: a copy of 1 KB
// into the LDS, a wait for its copies, a barrier, a pass through its epilogue region.  (tests/test_lds_copy_order.py builds
// this file, with the header's assembly statements turned into calls of sim_asm.)
//
//   lds_copy_order LAYOUT EPILOGUE K KEEP_H1 WORKERS rows...
//
// WORKERS workgroups share the items of one XCD; `rows` are the M tiles of its two pair slots (four numbers; 0: no tile).
// Output: per workgroup its first races and "races N"; at the end "copies N non-temporal M".
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#define __device__
#define __global__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define amdgpu_waves_per_eu(...) unused
struct Dim { unsigned x; };
static Dim threadIdx, blockIdx, gridDim;
using std::max;
using std::min;

struct Event { int kind, epoch, retired; uint32_t at; };   // retired: the wave's barriers when its wait let the copy pass
enum { kCopy, kEpilogue };
struct Wave { std::vector<Event> ev; std::vector<int> flight; int epoch = 0; };
static Wave waves[4];
static Wave* self;
static long n_copies[2];                                    // plain, non-temporal

static void sim_wait(int n) {
  auto& f = self->flight;                                   // in order; -1: a load into registers
  while ((int)f.size() > n) {
    if (f[0] >= 0) self->ev[f[0]].retired = self->epoch;
    f.erase(f.begin());
  }
}
static void sim_copy(uint32_t at, bool nt) {
  self->flight.push_back((int)self->ev.size());
  self->ev.push_back({kCopy, self->epoch, INT32_MAX, at});
  ++n_copies[nt];
}
static void sim_barrier() { ++self->epoch; }
static void sim_epilogue() { self->ev.push_back({kEpilogue, self->epoch, self->epoch, 0}); }

template <typename T> static long sim_num(const T& v) { if constexpr (std::is_integral_v<T>) return (long)v; else return 0; }
template <typename... A> static void sim_asm(const char* text, const A&... a) {
  const long v[] = {sim_num(a)..., 0, 0, 0, 0, 0};
  if (strstr(text, "global_load_lds")) sim_copy((uint32_t)(v[0] + (strstr(text, "s_add_u32") ? v[3] : 0)), strstr(text, " nt"));
  else if (strstr(text, "global_load")) self->flight.push_back(-1);
  else if (strstr(text, "s_waitcnt")) sim_wait((int)v[0]);
}

#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_readlane(x, l) (x)
#define __builtin_amdgcn_ballot_w64(p) ((uint64_t)(p))
#define __builtin_amdgcn_s_waitcnt(imm) sim_waitcnt(imm)
#define __builtin_amdgcn_s_barrier() sim_barrier()
#define __syncthreads() sim_barrier()
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() sim_epilogue()
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(p) (*(p))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_global_atomic_fadd_v2bf16(p, v) ((void)0)
static void sim_waitcnt(int imm) {
  const int vm = (imm & 15) | ((imm >> 14) & 3) << 4;
  if (vm < 63) sim_wait(vm);
}
extern "C" __attribute__((weak)) __bf16 __truncsfbf2(float) { return __builtin_bit_cast(__bf16, (uint16_t)0); }

#include "gemm_bf16.h"

namespace moe {
template <int LAY, int EPI>
void stream_gemm_bf16(const GemmParams&, int, char*) { abort(); }
}  // namespace moe
using namespace moe;

static std::vector<__bf16> g_out, g_h1;

template <int LAY, int EPI>
static void run(GemmParams p) {
  for (int w = 0; w < 4; ++w) {
    self = &waves[w];
    threadIdx.x = w * 64;
    grouped_gemm_bf16_kernel<LAY, EPI>(p);
    sim_wait(0);
  }
}

int main(int argc, char** argv) {
  const int lay = atoi(argv[1]), epi = atoi(argv[2]), K = atoi(argv[3]), keep_h1 = atoi(argv[4]), W = atoi(argv[5]);
  constexpr int kN = 512;
  // entries 0, 1 and 16, 17 of the map: the pair slots of XCD 0
  static int32_t expert[18], row0[18], rows[18], meta[kMetaWords], offsets[5];
  int n = 0;
  for (int i = 0; i < 4; ++i) {
    const int m = i < 2 ? i : 14 + i;
    rows[m] = i + 6 < argc ? atoi(argv[i + 6]) : 0;
    expert[m] = i;
    row0[m] = n;
    offsets[i] = n;
    n += rows[m];
  }
  offsets[4] = n;
  meta[kMetaMTiles] = 18; meta[kMetaMaxRows] = 1 << 20;
  g_out.resize((size_t)(n + 512) * 2 * kN); g_h1.resize((size_t)(n + 512) * 2 * kN);
  GemmParams p{};
  p.A = g_out.data(); p.B = g_out.data(); p.C = g_out.data();
  if (epi == kEpiSwiglu && keep_h1) p.C2 = g_h1.data();
  p.G = g_h1.data();
  p.N = kN; p.K = K; p.lda = K; p.ldc = 2 * kN; p.ldb = lay == kLayNT ? K : 2 * kN;
  p.n_ntiles = epi == kEpiSwiglu ? kN / 128 : kN / 256;
  p.offsets = offsets; p.E_local = 4; p.strideB = 1;
  p.tiles = TileMap{expert, row0, rows, meta};
  gridDim.x = 8 * W;
  for (int lw = 0; lw < W; ++lw) {
    for (Wave& w : waves) w = Wave();
    blockIdx.x = 8 * lw;
    if (lay == kLayNN && epi == kEpiSwiglu) run<kLayNN, kEpiSwiglu>(p);
    else if (lay == kLayNN) run<kLayNN, kEpiStore>(p);
    else if (epi == kEpiSwigluGrad) run<kLayNT, kEpiSwigluGrad>(p);
    else run<kLayNT, kEpiStore>(p);

    for (Wave& w : waves)
      if (w.epoch != waves[0].epoch) { printf("barriers differ\n"); return 1; }
    // the staging area starts where wave 0's first activation line goes
    uint32_t lds0 = 0;
    for (const Event& e : waves[0].ev) if (e.kind == kCopy) { lds0 = e.at; break; }
    int races = 0;
    char* const zero = nullptr;
    for (int a = 0; a < 4; ++a)
      for (const Event& x : waves[a].ev) {
        if (x.kind != kCopy) continue;
        const uint32_t lo = x.at - lds0;
        if (lo + kLine > (uint32_t)kGemmLdsBytes) { printf("copy outside the staging area\n"); return 1; }
        // the copy is complete for wave b once b is past the barrier that follows a's wait: b's epoch > x.retired
        for (int b = 0; b < 4; ++b) {
          if (b == a) continue;                              // a wave's own copies land in order, ahead of its epilogue
          const uint32_t reg = (uint32_t)(epilogue_region(zero, b) - zero);
          for (const Event& y : waves[b].ev) {
            const bool hit = y.kind == kCopy ? y.at == x.at : lo < reg + kEpiWaveBytes && reg < lo + kLine;
            if (!hit || y.epoch > x.retired || x.epoch > y.retired) continue;
            if (++races <= 3)
              printf("workgroup %d: wave %d copies to %u KB in interval %d (awaited in %d); wave %d %s in %d\n", lw, a, lo / 1024, x.epoch,
                     x.retired, b, y.kind == kCopy ? "copies there" : "has its epilogue there", y.epoch);
          }
        }
      }
    printf("races %d\n", races);
  }
  printf("copies %ld non-temporal %ld\n", n_copies[0] + n_copies[1], n_copies[1]);
  return 0;
}
