"""Order of the tiles of two weight gradients in one launch, on the CPU: csrc/wgrad_order.h as the device compiles it."""
import ctypes

import pytest

import host_build

pytestmark = pytest.mark.skipif(host_build.CXX is None, reason="needs a host C++ compiler")


@pytest.mark.parametrize("n0,n1", [(1, 0), (0, 1), (3, 3), (1, 4), (5, 2), (0, 6), (16, 16), (7, 256)])
@pytest.mark.parametrize("per0,per1", [(1, 1), (30, 54), (7, 1), (1, 9)])
def test_every_tile_once_and_experts_in_descending_rows(n0, per0, n1, per1):
    lib, out = host_build.library("wgrad_order.cpp"), (ctypes.c_int * 3)()
    seen, last = set(), 0
    for t in range(n0 * per0 + n1 * per1):
        lib.wgrad_pick(t, n0, per0, n1, per1, out)
        which, rank, tile = out
        assert which in (0, 1) and 0 <= rank < (n1 if which else n0) and 0 <= tile < (per1 if which else per0), (t, tuple(out))
        # the experts of either list are ranked by rows and the shorter list is the head of the longer one
        assert rank >= last, f"tile {t}: expert {rank} behind the smaller expert {last}"
        last = rank
        seen.add((which, rank, tile))
    assert len(seen) == n0 * per0 + n1 * per1


def test_one_gradient():
    """The launch of one gradient asks with an empty second one."""
    lib, out = host_build.library("wgrad_order.cpp"), (ctypes.c_int * 3)()
    for t in range(12):
        lib.wgrad_pick(t, 3, 4, 0, 0, out)
        assert tuple(out) == (0, t // 4, t % 4)
