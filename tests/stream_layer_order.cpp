// Runs the single launch of up to 64 tokens (csrc/stream_layer.h) on the CPU: every lane is a fiber, a scheduler decides which wave goes
// on, and the shares' arithmetic is replaced by a record of who ran which share when.  (tests/test_stream_layer_order.py builds this file
// beside a copy of the header whose own includes are empty.)
//
//   stream_layer_order POLICY SEED G RESIDENT T SPIN_LIMIT
//
// POLICY 0: any wave of a workgroup goes on; 1: wave 0 as long as it can; 2: wave 0 only when no other can.  RESIDENT workgroups are on
// the chip at a time.  Checked: all waves of a workgroup pass the same barriers; every share is run by one workgroup, with all of its
// waves; GEMM-2 starts behind all of GEMM-1's stores, Combine behind all of GEMM-2's; the launch ends; without expired waits every token
// is combined once.  Output: "combined N status S", or the first fault and exit status 1.
#include <ucontext.h>

#include <algorithm>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <random>
#include <type_traits>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(x)
#define __HIP_MEMORY_SCOPE_AGENT 0

struct Dim { int x; };
static Dim threadIdx, blockIdx, blockDim, gridDim;

namespace moe {
constexpr int kWave = 16, kNumXcd = 8, kWaves = 4;   // lanes beyond the eight classes, as on the device
constexpr int kGemmThreads = kWaves * kWave, kGemmLdsBytes = 256, kStreamBox = 64, kEvPerTile = 4, kMapSlack = 64;
enum { kMetaMaxRows = 0, kMetaRows = 1, kMetaStatus = 2, kMetaWords = 4 };
enum { kLayNN, kEpiStore, kEpiSwiglu, kStreamFirst, kStreamSecond };
struct GemmParams { const int32_t* offsets; const int32_t* gather; int E_local; };
struct PermuteParams {};
struct CombineParams { int T, H; };
}  // namespace moe

// ---- fibers ----
enum State { kReady, kBlocked, kEnded };
struct Lane { ucontext_t ctx; State state = kReady; std::unique_ptr<char[]> stack; };
struct WaveOf { std::vector<Lane> lanes{(size_t)moe::kWave}; int arrived = 0; long meeting = 0; uint32_t values[moe::kWave]; bool at_barrier = false; };
struct Group { WaveOf waves[moe::kWaves]; bool started = false, ended = false; int barrier_line = 0; char lds[moe::kGemmLdsBytes]; };
static std::vector<Group> groups;
static ucontext_t scheduler;
static int cur_group, cur_wave, cur_lane;
static std::mt19937 rng;

static void fault(const char* format, ...) {
  va_list args;
  va_start(args, format);
  printf("workgroup %d wave %d lane %d: ", cur_group, cur_wave, cur_lane);
  vprintf(format, args);
  printf("\n");
  exit(1);
}
static Group& group() { return groups[cur_group]; }
static WaveOf& wave_of() { return group().waves[cur_wave]; }
static Lane& lane_of() { return wave_of().lanes[cur_lane]; }
static void leave() {
  const int g = cur_group, w = cur_wave, l = cur_lane;
  swapcontext(&groups[g].waves[w].lanes[l].ctx, &scheduler);
}
static void block() { lane_of().state = kBlocked; leave(); }
static void wake(WaveOf& w) {
  for (Lane& l : w.lanes) if (l.state == kBlocked) l.state = kReady;
}

// All lanes of the wave meet.
static void meet() {
  WaveOf& w = wave_of();
  const long here = w.meeting;
  if (++w.arrived == moe::kWave) {
    w.arrived = 0;
    ++w.meeting;
    wake(w);
  }
  while (wave_of().meeting == here) block();
}
static uint32_t sim_readlane(uint32_t v, int from) {
  wave_of().values[cur_lane] = v;
  meet();
  const uint32_t r = wave_of().values[from];
  meet();
  return r;
}
static uint64_t sim_ballot(bool p) {
  wave_of().values[cur_lane] = p;
  meet();
  uint64_t m = 0;
  for (int i = 0; i < moe::kWave; ++i) m |= (uint64_t)(wave_of().values[i] != 0) << i;
  meet();
  return m;
}
static void sim_barrier(int line) {
  meet();
  Group& g = group();
  if (cur_lane == 0) {
    for (const WaveOf& w : g.waves)
      if (w.lanes[0].state == kEnded) fault("barrier in line %d, a wave has ended", line);
    int others = 0;
    for (const WaveOf& w : g.waves) others += w.at_barrier;
    if (others && g.barrier_line != line) fault("barrier in line %d, others in line %d", line, g.barrier_line);
    g.barrier_line = line;
    wave_of().at_barrier = true;
    if (others + 1 == moe::kWaves)
      for (WaveOf& w : g.waves) { w.at_barrier = false; wake(w); }
    while (wave_of().at_barrier) block();
  }
  meet();
}

#define __syncthreads() sim_barrier(__LINE__)
#define __ballot(p) sim_ballot(p)
#define __builtin_amdgcn_readfirstlane(x) ((int)sim_readlane((uint32_t)(x), 0))
#define __builtin_amdgcn_readlane(x, l) ((int)sim_readlane((uint32_t)(x), l))
#define __builtin_amdgcn_s_sleep(x) leave()
#define __builtin_amdgcn_fence(...) ((void)0)
template <typename T, typename V> static T sim_add(T* p, V v) { leave(); const T old = *p; *p += v; leave(); return old; }
template <typename T> static T sim_load(const T* p) { leave(); const T v = *p; leave(); return v; }
#define __hip_atomic_fetch_add(p, v, order, scope) sim_add(p, v)
#define __hip_atomic_load(p, order, scope) sim_load(p)
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))

// ---- what the launch calls ----
static int stored[2][512], runner[2][512];   // per share: waves whose results are in memory; the workgroup that runs it, -1
static int combined[256], copied[256];
namespace moe {
using std::min;
static int lane_id() { return cur_lane; }
static void wait_own_stores() {}
static uint32_t wave_atomic_add(uint32_t* p, uint32_t inc) {
  uint32_t old = 0;
  if (cur_lane == 0) old = sim_add(p, inc);
  return sim_readlane(old, 0);
}
static int stream_tables(const int32_t*, int, const int32_t*, char*) { __syncthreads(); return 1; }
static void all_stored(int gemm) {
  for (int v = 0; v < gridDim.x; ++v)
    if (stored[gemm][v] != kWaves) fault("reads results of GEMM-%d whose share %d is stored by %d waves", gemm + 1, v, stored[gemm][v]);
}
template <int LAY, int EPI, int ROLE, typename Ready>
static void stream_share(const GemmParams&, int, int, int v, char*, Ready&& ready) {
  constexpr int gemm = ROLE == kStreamSecond;
  if (v < 0 || v >= gridDim.x) fault("share %d of GEMM-%d", v, gemm + 1);
  if (runner[gemm][v] >= 0 && runner[gemm][v] != cur_group) fault("share %d of GEMM-%d again", v, gemm + 1);
  runner[gemm][v] = cur_group;
  if (gemm) {
    if (!ready()) return;
    all_stored(0);
  }
  for (int i = (int)(v * 7 % 13); i > 0; --i) leave();
  meet();
  if (cur_lane == 0 && ++stored[gemm][v] > kWaves) fault("share %d of GEMM-%d again", v, gemm + 1);
  __syncthreads();
}
template <int U>
static void permute_rows(const PermuteParams&, int r0, int r1, int wave, int n_waves) {
  if (cur_lane == 0) for (int r = r0 + wave; r < r1; r += n_waves) ++copied[r];
}
static void combine_load_slots(const CombineParams&, int, int& rowv, float& wv) { rowv = 0; wv = 0.0f; }
template <bool BF16, int U, int N>
static void combine_token_rows(const CombineParams&, int t, int, float) {
  all_stored(1);
  if (cur_lane == 0) ++combined[t];
}
template <typename F> static void with_row_vectors(int, F&& f) { f(std::integral_constant<int, 4>{}); }
}  // namespace moe

#include "stream_layer.h"

static moe::StreamLayerParams params;
static void lane_main() {
  moe::stream_layer_kernel(params);
  lane_of().state = kEnded;
  for (;;) leave();
}

// Every lane of the wave that can goes on once.
static void step(int g, int w) {
  for (int l = 0; l < moe::kWave; ++l) {
    Lane& lane = groups[g].waves[w].lanes[l];
    if (lane.state != kReady) continue;
    cur_group = g; cur_wave = w; cur_lane = l;
    blockIdx.x = g; threadIdx.x = w * moe::kWave + l;
    swapcontext(&scheduler, &lane.ctx);
  }
}
static bool can(const WaveOf& w) {
  for (const Lane& l : w.lanes) if (l.state == kReady) return true;
  return false;
}
static bool over(const WaveOf& w) {
  for (const Lane& l : w.lanes) if (l.state != kEnded) return false;
  return true;
}

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  const int policy = atoi(argv[1]), G = atoi(argv[3]), resident = atoi(argv[4]), T = atoi(argv[5]);
  rng.seed((unsigned)atoi(argv[2]));
  constexpr int kRows = 100;
  static uint32_t events[moe::kStreamLayerEvents];
  static int32_t meta[moe::kMetaWords] = {1, kRows, 0, 0};
  memset(runner, -1, sizeof(runner));
  params.comb = {T, 64};
  params.events = events; params.meta = meta;
  params.copy = 1;
  params.spin_limit = (uint32_t)strtoul(argv[6], nullptr, 0);
  params.timeout_status = -5;
  gridDim.x = G; blockDim.x = moe::kGemmThreads;
  groups = std::vector<Group>(G);
  for (Group& g : groups)
    for (WaveOf& w : g.waves)
      for (Lane& l : w.lanes) {
        constexpr size_t kStack = 32 * 1024;
        l.stack.reset(new char[kStack]);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.get();
        l.ctx.uc_stack.ss_size = kStack;
        makecontext(&l.ctx, lane_main, 0);
      }
  std::vector<int> live;
  int next = 0;
  long idle = 0;
  for (long steps = 0;; ++steps) {
    while ((int)live.size() < resident && next < G && (live.empty() || rng() % 64 == 0)) live.push_back(next++);
    if (live.empty()) break;
    const size_t at = rng() % live.size();
    Group& g = groups[live[at]];
    int w = (int)(rng() % moe::kWaves);
    if (policy == 1) { if (can(g.waves[0])) w = 0; }
    else if (policy == 2) { if (w == 0 && (can(g.waves[1]) || can(g.waves[2]) || can(g.waves[3]))) w = 1 + (int)(rng() % 3); }
    if (can(g.waves[w])) { step(live[at], w); idle = 0; }
    else if (++idle > 100000) { printf("nothing goes on\n"); return 1; }
    if (steps > 50000000) { printf("the launch does not end\n"); return 1; }
    bool done = true;
    for (const WaveOf& x : g.waves) done = done && over(x);
    if (done) live.erase(live.begin() + (long)at);
  }
  cur_group = cur_wave = cur_lane = -1;
  int n = 0;
  for (int t = 0; t < T; ++t) {
    if (combined[t] > 1) fault("token %d combined %d times", t, combined[t]);
    n += combined[t];
  }
  if (meta[moe::kMetaStatus] == 0) {
    if (n != T) fault("%d of %d tokens combined, no status", n, T);
    for (int gemm = 0; gemm < 2; ++gemm) moe::all_stored(gemm);
  }
  for (int r = 0; r < kRows; ++r) if (copied[r] != 1) fault("row %d copied %d times", r, copied[r]);
  printf("combined %d status %d\n", n, meta[moe::kMetaStatus]);
  return 0;
}
