"""Choice of form of the weight stream, on the CPU: csrc/stream_rule.h as the device compiles it, over every launch it takes."""
import pytest

import stream_rule

pytestmark = pytest.mark.skipif(stream_rule.CXX is None, reason="needs a host C++ compiler")


@pytest.mark.parametrize("G", [8, 248, 256, 304])
def test_every_form_holds_its_launch(G):
    """Rows of a stage >= rows of the largest expert, items that cover the columns once, a form that the kernel has."""
    n, first = stream_rule.faults(G)
    assert n == 0, f"{n} launches, one of them (max_rows, experts with rows, N, swiglu) = {first}: {stream_rule.form(*first, G)}"


@pytest.mark.parametrize("G", [248, 256, 304])
def test_no_form_makes_rounds_longer(G):
    """A round costs its columns: no workgroup has more of them than with 128 columns per item throughout."""
    n, first = stream_rule.longer(G)
    assert n == 0, f"{n} launches, one of them (max_rows, experts with rows, N, swiglu) = {first}: {stream_rule.form(*first, G)}"


@pytest.mark.parametrize("N,n_act", [(64, 160), (192, 70), (320, 48), (448, 35), (576, 27), (704, 22), (832, 19), (960, 17), (1088, 15),
                                     (1216, 13), (1344, 12), (1472, 11), (1600, 10), (3264, 5)])
def test_stages_of_128_rows_above_64_rows(N, n_act):
    """One round of 128-column items whose 256-column items would be more than half a round: N / 64 is odd."""
    for max_rows in (65, 128):
        assert stream_rule.form(max_rows, n_act, N, True, 256)[:2] == (128, 128)
    assert stream_rule.form(129, n_act, N, True, 256) is None
