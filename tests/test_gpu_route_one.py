"""Routing of few tokens in one launch (up to 64) and of the next size in two: every number of experts per lane (the steps of
the selection: 16, 32, 64, 128, 256 experts), the edges of the 64-token mask, shards, ties.  Integers are exact, the routing
weights those of the other routing tests; the tile scheduler runs on the tables of the same launch (bit-equal output)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 5, 63, 64, 65])
@pytest.mark.parametrize("E,E_local,base,k", [(1, 1, 0, 1), (16, 16, 0, 16), (17, 5, 9, 3), (32, 32, 0, 4), (33, 7, 26, 8), (64, 64, 0, 8),
                                              (66, 1, 65, 2), (128, 100, 20, 16), (130, 130, 0, 5), (256, 256, 0, 8), (256, 65, 191, 16)])
def test_routing_of_few_tokens(T, E, E_local, base, k):
    from gpu_common import check_forward, check_routing, run_forward, small_config
    cfg = small_config("route_one", T, 64, 64, E, E_local, base, k, "bf16", 91)
    inp = make_inputs(cfg)
    inp["logits"][:] = np.round(inp["logits"] * 2) / 2     # many ties: the lowest expert first
    inp["logits"][0, ::3] = -0.0
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], k, base, E_local)
    run = run_forward(cfg, inp)
    check_routing(run, ref)
    if ref["counts"].sum():
        check_forward(run, ref, "bf16")
    else:
        assert torch.all(run.out == 0)
    single = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT)
    check_routing(single, ref)
    assert torch.equal(single.out, run.out)
