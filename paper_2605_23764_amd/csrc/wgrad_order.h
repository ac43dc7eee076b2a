// Order of the tiles of a launch with two weight gradients (wgrad_bf16.h), kept free of device code so that a test on the host
// can go through it (tests/wgrad_order.cpp).
#pragma once

namespace moe {

struct WgradPick {
  int which;   // gradient 0 or 1
  int rank;    // place of the expert in the list, most rows first
  int tile;    // of the expert's tiles in that gradient
};

// Tile t of n0 experts with per0 tiles each in gradient 0 and n1 with per1 in gradient 1.  Both lists start with the same experts
// in the same order (each holds all experts from some number of rows on, most rows first).  An expert's tiles of both gradients
// stand side by side, so that the whole list descends in rows: a sweep is balanced and the last one holds the cheapest tiles.
// With gradient 1's list behind the whole of gradient 0's, a sweep had gradient 0's smallest experts beside gradient 1's largest:
// backward, skewed routing, T = 4096, H = 1088, I = 704, 16 experts, k = 4 405 us against 348; T = 8192, 32 experts 702 and 624;
// H = 2048, I = 1408 840 and 799; H = 2112, I = 1472, T = 2000 557 and 561; even routing level.
constexpr WgradPick wgrad_pick(int t, int n0, int per0, int n1, int per1) {
  const int both = n0 < n1 ? n0 : n1, per = per0 + per1;
  if (t < both * per) {
    const int rank = t / per, tile = t - rank * per;
    return tile < per0 ? WgradPick{0, rank, tile} : WgradPick{1, rank, tile - per0};
  }
  const int which = n1 > n0, p = which ? per1 : per0, rest = t - both * per, rank = rest / p;
  return {which, both + rank, rest - rank * p};
}

}  // namespace moe
