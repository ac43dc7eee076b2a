// The choice of form of the weight stream (csrc/stream_rule.h), built for the host by tests/stream_rule.py.
#include "stream_rule.h"

extern "C" int stream_takes(int max_rows, int n_act, int N, int swiglu, int G) { return moe::stream_takes(max_rows, n_act, N, swiglu, G); }

// form: {columns per item, rows of a stage, items, whole items}
extern "C" void stream_form(int max_rows, int n_act, int N, int swiglu, int G, int* form) {
  const moe::StreamForm f = moe::stream_form(max_rows, n_act, N, swiglu, G);
  form[0] = f.cols; form[1] = f.rows; form[2] = f.items; form[3] = f.whole;
}

// Every launch with N = 64, 128 .. 8192 and 1..256 experts that the stream takes: returns how many have a form that does not
// hold the rows, does not cover the columns exactly once or that the kernel doesn't have; `first` is one of them.
extern "C" int stream_faults(int G, int* first) {
  int n = 0;
  for (int swiglu = 0; swiglu < 2; ++swiglu)
    for (int N = 64; N <= 8192; N += 64)
      for (int n_act = 1; n_act <= 256; ++n_act)
        for (int max_rows = 1; max_rows <= 130; ++max_rows) {
          if (!moe::stream_takes(max_rows, n_act, N, swiglu, G)) continue;
          const moe::StreamForm f = moe::stream_form(max_rows, n_act, N, swiglu, G);
          const int out = swiglu ? f.cols / 2 : f.cols, per = (N + out - 1) / out;
          bool ok = f.rows >= max_rows && f.items == n_act * per;
          if (f.cols == 64) ok &= f.items <= G && f.whole == f.items && (f.rows == 16 || f.rows == 32 || f.rows == 64 || f.rows == 128);
          else if (f.cols == 128) ok &= f.whole == f.items && (f.rows == 32 || f.rows == 64 || f.rows == 128);
          else ok &= f.cols == 256 && swiglu && (f.rows == 32 || f.rows == 64) && f.whole >= 0 && f.whole <= f.items &&
                     (f.whole == f.items || N % out == 0);   // a rest as halves: both halves of every item have columns
          if (!ok && n++ == 0) { first[0] = max_rows; first[1] = n_act; first[2] = N; first[3] = swiglu; }
        }
  return n;
}

// Launches of at most 64 rows in which some workgroup gets more columns than with 128 columns per item throughout.
extern "C" int stream_longer(int G, int* first) {
  auto rounds = [&](int items) { return (items + G - 1) / G; };
  int n = 0;
  for (int swiglu = 0; swiglu < 2; ++swiglu)
    for (int N = 64; N <= 8192; N += 64)
      for (int n_act = 1; n_act <= 256; ++n_act)
        for (int max_rows = 1; max_rows <= moe::kStreamRows; ++max_rows) {
          const moe::StreamForm f = moe::stream_form(max_rows, n_act, N, swiglu, G);
          const int out128 = swiglu ? 64 : 128, by128 = 128 * rounds(n_act * ((N + out128 - 1) / out128));
          if (f.cols * rounds(f.whole) + 128 * rounds(2 * (f.items - f.whole)) <= by128) continue;
          if (n++ == 0) { first[0] = max_rows; first[1] = n_act; first[2] = N; first[3] = swiglu; }
        }
  return n;
}
