// A launch on the CPU: every lane is a fiber, a scheduler decides which wave goes on.  Included ahead of a kernel's header.
// POLICY 0: any wave of a workgroup goes on; 1: wave 0 as long as it can; 2: wave 0 only when no other can.
#pragma once
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
constexpr int kGemmThreads = kWaves * kWave, kGemmLdsBytes = 256;
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
static void (*lane_kernel)();

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

namespace moe {
using std::max;
using std::min;
static int lane_id() { return cur_lane; }
static void wait_own_stores() {}
static uint32_t wave_atomic_add(uint32_t* p, uint32_t inc) {
  uint32_t old = 0;
  if (cur_lane == 0) old = sim_add(p, inc);
  return sim_readlane(old, 0);
}
}  // namespace moe

static void lane_main() {
  lane_kernel();
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


// A launch of G workgroups, RESIDENT of them on the chip at a time.  A fault ends the program with status 1.
static void run_launch(void (*kernel)(), int policy, int seed, int G, int resident) {
  rng.seed((unsigned)seed);
  lane_kernel = kernel;
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
    else if (++idle > 100000) { printf("nothing goes on\n"); exit(1); }
    if (steps > 50000000) { printf("the launch does not end\n"); exit(1); }
    bool done = true;
    for (const WaveOf& x : g.waves) done = done && over(x);
    if (done) live.erase(live.begin() + (long)at);
  }
  cur_group = cur_wave = cur_lane = -1;
}
