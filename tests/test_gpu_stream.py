"""Grouped GEMMs as a weight stream (largest expert of at most 64 rows): the edges of its shapes, against the fp64 oracle
and bit for bit against the single launch, which runs the same products through the ordinary tiles (both sum K in the
same order)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # name, H, I, rows per expert (repeated over the experts)
    ("one_row", 128, 64, [1, 0, 0]),                        # one expert; 64 columns per item, a single stage
    ("narrow_16", 320, 192, [16, 1, 0, 9]),                 # 16-row stages; K = 2.5 and 1.5 stages of 128
    ("narrow_32", 192, 320, [17, 32, 3]),                   # 32-row stages with 64 columns
    ("wide_32", 448, 832, [32, 2, 31, 0] * 12),             # 128 columns, several items per workgroup, N = 3.5 and 6.5 tiles
    ("wide_64", 320, 448, [64, 33, 1, 0, 50]),              # two row blocks
    ("many_rows", 128, 192, [40] * 64),                     # more rows than the token table in LDS holds
    ("above", 192, 128, [65, 3]),                           # the first size that takes the ordinary tiles
]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_weight_stream(case, keep_xp):
    from gpu_common import check_backward, check_forward, check_routing, run_backward, run_forward, small_config
    name, H, I, rows = case
    E = len(rows)
    cfg = small_config("stream_" + name, sum(rows), H, I, E, E, 0, 1, "bf16", 81)
    inp = make_inputs(cfg, with_dy=True)
    inp["logits"][:] = -10.0
    inp["logits"][np.arange(cfg.T), np.random.default_rng(4).permutation(np.repeat(np.arange(E), rows))] = 1.0
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k)
    assert ref["counts"].tolist() == rows
    run = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
    check_routing(run, ref)
    check_forward(run, ref, "bf16", store_h1=True)
    single = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True, keep_xp=keep_xp)
    for n in ("A", "H1", "Yp"):
        assert torch.equal(getattr(single.saved, n)[:cfg.T], getattr(run.saved, n)[:cfg.T]), n
    assert torch.equal(single.out, run.out)
    bwd, bwd_single = run_backward(cfg, inp, run), run_backward(cfg, inp, run, mode=moe.MODE_PERSISTENT)
    check_backward(bwd, oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"]), ref["counts"], "bf16")
    assert torch.equal(bwd.dx, bwd_single.dx) and torch.equal(bwd.dw_gate_up, bwd_single.dw_gate_up)
