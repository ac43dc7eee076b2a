// Runs the single launch of up to 64 tokens (csrc/stream_layer.h) on the CPU (fibers.h); the shares' arithmetic is replaced by a record of
// who ran which share when.  (tests/test_stream_layer_order.py builds this file beside a copy of the header whose own includes are empty.)
//
//   stream_layer_order POLICY SEED G RESIDENT T SPIN_LIMIT
//
// Checked: all waves of a workgroup pass the same barriers; every share is run by one workgroup, with all of its
// waves; GEMM-2 starts behind all of GEMM-1's stores, Combine behind all of GEMM-2's; the launch ends; without expired waits every token
// is combined once.  Output: "combined N status S", or the first fault and exit status 1.
#include "fibers.h"

// ---- what the launch calls ----
static int stored[2][512], runner[2][512];   // per share: waves whose results are in memory; the workgroup that runs it, -1
static int combined[256], copied[256];
namespace moe {
constexpr int kStreamBox = 64, kEvPerTile = 4, kMapSlack = 64;
enum { kMetaMaxRows = 0, kMetaRows = 1, kMetaStatus = 2, kMetaWords = 4 };
enum { kLayNN, kEpiStore, kEpiSwiglu, kStreamFirst, kStreamSecond };
struct GemmParams { const int32_t* offsets; const int32_t* gather; int E_local; };
struct PermuteParams {};
struct CombineParams { int T, H; };
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
int main(int argc, char** argv) {
  if (argc != 7) return 2;
  const int policy = atoi(argv[1]), G = atoi(argv[3]), resident = atoi(argv[4]), T = atoi(argv[5]);
  constexpr int kRows = 100;
  static uint32_t events[moe::kStreamLayerEvents];
  static int32_t meta[moe::kMetaWords] = {1, kRows, 0, 0};
  memset(runner, -1, sizeof(runner));
  params.comb = {T, 64};
  params.events = events; params.meta = meta;
  params.copy = 1;
  params.spin_limit = (uint32_t)strtoul(argv[6], nullptr, 0);
  params.timeout_status = -5;
  run_launch([] { moe::stream_layer_kernel(params); }, policy, atoi(argv[2]), G, resident);
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
