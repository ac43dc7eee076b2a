// Which grouped bf16 GEMMs run as a weight stream, and in which form: arithmetic on words that the device reads from the tile
// map, kept free of device code so that a test on the host goes through all of it (tests/stream_rule.cpp).
#pragma once

namespace moe {

constexpr int kStreamRows = 64;       // rows of the largest expert up to which a launch runs as a weight stream,
constexpr int kStreamMaxRows = 128;   // ... and up to which it does where that takes a single round (stream_takes)

constexpr int stream_tiles(int n, int per) { return (n + per - 1) / per; }

// A launch of G workgroups over N output columns (swiglu: of gate and up, an item's columns are half of either) of n_act experts
// with rows, max_rows in the largest.
//
// 65..128 rows per expert: as a stream where its items of 128 columns are a single round, i.e. where tiles of 256 columns
// leave half of the chip idle (T = 777, H = 1088, I = 704, 10 experts: training step 133 -> 115 us; 1600 rows, H = 7168,
// I = 512, 4 experts: forward 141 -> 96, backward 212 -> 159; T = 400, H = 2048, I = 1408, 16 experts: gate_grad and act_grad,
// backward 206 -> 194).  With more items than workgroups the tiles win (the same layer's GEMM-1: forward 95 as tiles, 106 as
// a stream; H = 7168, I = 2048, 32 experts: 603 and 669), and above 128 rows too (150 rows, 16 experts: 54 and 60).
constexpr bool stream_takes(int max_rows, int n_act, int N, bool swiglu, int G) {
  return max_rows <= kStreamRows || (max_rows <= kStreamMaxRows && n_act * stream_tiles(N, swiglu ? 64 : 128) <= G);
}

struct StreamForm {
  int cols;    // weight columns per item: 64, 128 or 256
  int rows;    // activation rows that a stage holds, for every form at least max_rows
  int items;   // items of `cols` columns
  int whole;   // the first of them, which run as such; the others run as two of 128 columns each
};

constexpr StreamForm stream_form(int max_rows, int n_act, int N, bool swiglu, int G) {
  // 128 columns per item; 64 only where that still is a single round, i.e. where the chip would be at most half full
  // (T = 1, H = 2048, I = 1408, four experts: GEMM-1 88 items -> 176): 64 columns are 128-byte pieces of a row, 64-byte
  // pieces for SwiGLU (half gate, half up), which stream 10..30 % slower once all CUs are busy (T = 64: 84 us a layer
  // against 73).
  const int n64 = n_act * stream_tiles(N, swiglu ? 32 : 64), n128 = n_act * stream_tiles(N, swiglu ? 64 : 128);
  if (n64 <= G) return {64, max_rows <= 16 ? 16 : max_rows <= 32 ? 32 : max_rows <= 64 ? 64 : 128, n64, n64};
  // GEMM-1: 256 columns (128 gate, 128 up: 256-byte pieces instead of 128; T = 256, H = 7168 515 -> 475 us a layer, T = 64,
  // H = 2048 73 -> 67).  Where that leaves a last round at most half full, its items run as two of 128 columns each: a round
  // costs its columns, and whole rounds keep the longer pieces (about 20 experts with rows, 320 items on 256 workgroups: T = 32
  // 350 us a layer with 128 columns throughout, 328 so; T = 24 318 -> 295; 32 experts, H = 4096, I = 1536, T = 64 224 -> 210).
  // A stage of this form holds 64 rows.
  if (swiglu && max_rows <= kStreamRows) {
    const int n256 = n_act * stream_tiles(N, 128), rest = n256 % G;
    if (2 * rest > G || rest == 0 || (n256 > G && N % 128 == 0))
      return {256, max_rows <= 32 ? 32 : 64, n256, 2 * rest > G ? n256 : n256 - rest};
  }
  return {128, max_rows <= 32 ? 32 : max_rows <= 64 ? 64 : 128, n128, n128};
}

}  // namespace moe
