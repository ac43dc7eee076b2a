// The order of the tiles of two weight gradients in one launch (csrc/wgrad_order.h), built for the host by tests/host_build.py.
#include "wgrad_order.h"

extern "C" void wgrad_pick(int t, int n0, int per0, int n1, int per1, int* out) {
  const moe::WgradPick p = moe::wgrad_pick(t, n0, per0, n1, per1);
  out[0] = p.which; out[1] = p.rank; out[2] = p.tile;
}
