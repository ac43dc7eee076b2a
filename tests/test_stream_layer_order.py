"""Order of the single launch of up to 64 tokens, on the CPU: csrc/stream_layer.h itself is compiled for the host with a fiber per lane
(tests/stream_layer_order.cpp) and run under schedules in which waves run ahead of or behind each other, workgroups start late and only
some of them fit on the chip."""
import os
import subprocess

import pytest

from host_build import CSRC, CXX, HERE

pytestmark = pytest.mark.skipif(CXX is None, reason="needs a host C++ compiler")


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    d = tmp_path_factory.mktemp("stream_layer_order")
    for name in ("gemm_stream.h", "permute_combine.h", "persistent.h", "wave_sync.h"):
        (d / name).write_text("#pragma once\n")
    with open(os.path.join(CSRC, "stream_layer.h")) as f:
        src = f.read()
    shared = "__shared__ __attribute__((aligned(1024))) char smem[kGemmLdsBytes];"
    assert src.count(shared) == 1
    (d / "stream_layer.h").write_text(src.replace(shared, "char* const smem = group().lds;"))
    exe = str(d / "stream_layer_order")
    res = subprocess.run([CXX, "-std=c++17", "-O1", "-w", "-I", str(d), "-I", HERE, os.path.join(HERE, "stream_layer_order.cpp"), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def run(policy, seed, G, resident, T, spin_limit=1 << 30):
        res = subprocess.run([exe, *map(str, (policy, seed, G, resident, T, spin_limit))], capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, ((policy, seed, G, resident, T, spin_limit), res.stdout + res.stderr)
        _, n, _, status = res.stdout.split()
        return int(n), int(status)

    return run


@pytest.mark.parametrize("G,resident", [(8, 8), (16, 16), (16, 7), (24, 3), (16, 1)])
@pytest.mark.parametrize("policy", [0, 1, 2], ids=["any_wave", "wave_0_ahead", "wave_0_behind"])
def test_every_share_once_under_any_schedule(sim, policy, G, resident):
    for seed in range(6):
        T = (1, 5, G, 64)[seed % 4]
        assert sim(policy, seed, G, resident, T) == (T, 0)


@pytest.mark.parametrize("spin_limit", [0, 1, 20])
@pytest.mark.parametrize("policy", [0, 1, 2], ids=["any_wave", "wave_0_ahead", "wave_0_behind"])
def test_expired_wait_combines_only_stored_rows(sim, policy, spin_limit):
    """(The simulation fails where a token is combined while a share of GEMM-2 is not stored.)  Without polls, and with workgroups that
    end before others start, GEMM-2 gives up somewhere: nothing is combined."""
    for seed in range(8):
        for G, resident in ((8, 8), (16, 16), (16, 7)):
            n, status = sim(policy, seed, G, resident, 64, spin_limit)
            assert status == -5 or n == 64
            if spin_limit == 0:
                assert (n, status) == (0, -5)
