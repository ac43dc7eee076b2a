// Which grouped bf16 GEMMs run as a weight stream, and in which form: arithmetic on words that the device reads from the tile
// map, kept free of device code so that a test on the host goes through all of it (tests/stream_rule.cpp).
#pragma once

// Inlined ahead of all optimization: as ordinary functions, inlined late, they left the grouped GEMM kernels with other registers
// at their head, and launches of a few rows took 0.5 us more (T = 777, H = 1088, I = 704, 10 experts, training step 106.9 us
// against 106.1).  The kernels' time follows such details: of eight ways to write the same choice the slowest cost skewed layers
// of T = 152..220 (H = 2048, I = 1408, 16 experts) 3 % of 85..90 us with K loops instruction for instruction the same.
#define MOE_RULE __attribute__((always_inline)) constexpr

namespace moe {

constexpr int kStreamRows = 64;       // rows of the largest expert up to which a launch runs as a weight stream,
constexpr int kStreamMaxRows = 128;   // ... and up to which it does where that takes a single round (stream_takes)

MOE_RULE int stream_tiles(int n, int per) { return (n + per - 1) / per; }

// A launch of G workgroups over N output columns (swiglu: of gate and up, an item's columns are half of either) of n_act experts
// with rows, max_rows in the largest.
//
// 65..128 rows per expert: as a stream where its items of 128 columns are a single round, i.e. where tiles of 256 columns
// leave half of the chip idle, with an odd N / 64 a little less (19 experts, I = 832: 133 tiles on 256 CUs).  T = 777, H = 1088,
// I = 704, 10 experts: training step 133 -> 115 us; 1600 rows, H = 7168, I = 512, 4 experts: forward 141 -> 96, backward
// 212 -> 159; T = 400, H = 2048, I = 1408, 16 experts: gate_grad and act_grad, backward 206 -> 194; T = 550, H = 1024, I = 704,
// 22 experts: training step 170 -> 157.  With more items than workgroups the tiles win (GEMM-1 of the layer of T = 400: forward 95
// as tiles, 106 as a stream; H = 7168, I = 2048, 32 experts: 603 and 669), and above 128 rows too (150 rows, 16 experts: 54 and 60).
MOE_RULE bool stream_takes(int max_rows, int n_act, int N, bool swiglu, int G) {
  return max_rows <= kStreamRows || (max_rows <= kStreamMaxRows && n_act * stream_tiles(N, swiglu ? 64 : 128) <= G);
}

// 128 columns per item; 64 only where that still is a single round, i.e. where the chip would be at most half full
// (T = 1, H = 2048, I = 1408, four experts: GEMM-1 88 items -> 176): 64 columns are 128-byte pieces of a row, 64-byte
// pieces for SwiGLU (half gate, half up), which stream 10..30 % slower once all CUs are busy (T = 64: 84 us a layer
// against 73).
MOE_RULE bool stream_narrow(int n_act, int N, bool swiglu, int G) { return n_act * stream_tiles(N, swiglu ? 32 : 64) <= G; }

// GEMM-1: 256 columns (128 gate, 128 up: 256-byte pieces instead of 128; T = 256, H = 7168 515 -> 475 us a layer, T = 64,
// H = 2048 73 -> 67) where no workgroup gets more columns that way than with 128 throughout: a round costs its columns.  Where a
// last round of at most half the workgroups is the reason that one would, its items run as two of 128 columns each behind the
// whole rounds (about 20 experts with rows, 320 items on 256 workgroups: T = 32 350 us a layer with 128 columns throughout, 328 so;
// T = 24 318 -> 295; 32 experts, H = 4096, I = 1536, T = 64 224 -> 210).  Otherwise (less than one round; N / 64 odd, where every
// expert's last item is half empty) 128 throughout.  256 columns there took, H = 2048, 35 rows an expert, I = 1600: 10 experts 69.6
// us a layer against 60.7, 30 experts 138.0 and 133.6; I = 704, 22 experts 73.2 and 64.9; 8 rows an expert 2..10 % more.  Only four
// rounds against seven and more than 32 rows went the other way, by 1 % (I = 1984, 57 experts 287.0 and 289.4).
// A stage of this form holds 64 rows.  n256, n128: the launch's items of either width.
MOE_RULE bool stream_wide_throughout(int n256, int n128, int G) {
  // 2 * ceil(n256 / G) <= ceil(n128 / G), from the last round's items and the 128-column halves that have no columns
  const int rest = n256 % G, missing = 2 * n256 - n128;
  return 2 * (rest ? rest : G) - missing > G;
}
MOE_RULE bool stream_wide(int max_rows, int n256, int n128, int N, int G) {
  return max_rows <= kStreamRows && (stream_wide_throughout(n256, n128, G) || (n256 > G && N % 128 == 0));
}
// Items that run with 256 columns; the others as two of 128 each.
MOE_RULE int stream_whole(int n256, int n128, int G) { return stream_wide_throughout(n256, n128, G) ? n256 : n256 - n256 % G; }

// Activation rows that a stage holds, for every form at least max_rows.
MOE_RULE int stream_stage_rows(int cols, int max_rows) {
  return cols == 64 && max_rows <= 16 ? 16 : max_rows <= 32 ? 32 : cols == 256 || max_rows <= 64 ? 64 : 128;
}

// All of it, as stream_gemm_bf16 puts it together.
struct StreamForm {
  int cols;    // weight columns per item: 64, 128 or 256
  int rows;    // activation rows that a stage holds
  int items;   // items of `cols` columns
  int whole;   // the first of them, which run as such; the others run as two of 128 columns each
};
MOE_RULE StreamForm stream_form(int max_rows, int n_act, int N, bool swiglu, int G) {
  const int n64 = n_act * stream_tiles(N, swiglu ? 32 : 64), n128 = n_act * stream_tiles(N, swiglu ? 64 : 128);
  const int n256 = n_act * stream_tiles(N, 128);
  if (stream_narrow(n_act, N, swiglu, G)) return {64, stream_stage_rows(64, max_rows), n64, n64};
  if (swiglu && stream_wide(max_rows, n256, n128, N, G)) return {256, stream_stage_rows(256, max_rows), n256, stream_whole(n256, n128, G)};
  return {128, stream_stage_rows(128, max_rows), n128, n128};
}

}  // namespace moe

#undef MOE_RULE
