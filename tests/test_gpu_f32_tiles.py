"""fp32 grouped GEMMs on the matrix pipe at the edges of their tiles: 64 rows (two wave rows of 32), 64 columns, a
reduction in steps of 16 that the weight gradients cut at an expert's last row.  Against the fp64 oracle; the bound is
the fp32 one of the other tests (1e-5 of the largest element; sums of at most 320 products)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# rows per expert: none, one, around 16, 32 and 64, and three tiles
ROWS = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130]


@pytest.mark.parametrize("H,I,keep_xp", [(64, 64, True), (320, 192, False)])
def test_edges_of_the_fp32_tiles(H, I, keep_xp):
    from gpu_common import check_backward, check_forward, check_routing, run_backward, run_forward, small_config
    cfg = small_config("f32_edges", sum(ROWS), H, I, len(ROWS), len(ROWS), 0, 1, "f32", 71)
    inp = make_inputs(cfg, with_dy=True)
    inp["logits"][:] = -10.0
    inp["logits"][np.arange(cfg.T), np.random.default_rng(3).permutation(np.repeat(np.arange(len(ROWS)), ROWS))] = 1.0
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k)
    assert ref["counts"].tolist() == ROWS
    run = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
    check_routing(run, ref)
    check_forward(run, ref, "f32", store_h1=True)
    single = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True, keep_xp=keep_xp)
    assert torch.equal(single.out, run.out)
    check_backward(run_backward(cfg, inp, run), oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"]), ref["counts"], "f32")


# up to 16 rows per expert: GEMM-1 133 and GEMM-2 152 strips of 64 columns (above 128), of 3 experts 21 and 24 tiles as two
# quarters each; up to 32 rows two quarters per tile, above that four
@pytest.mark.parametrize("rows", [[16, 1, 9, 15] * 4 + [2, 16, 0, 8], [16, 3, 1], [17, 32, 1, 0, 30] * 4, [33, 2, 16]])
def test_few_rows(rows):
    _whole_tiles_and_quarters("f32_few_rows", 512, 448, rows)


# 66 M tiles by 16 column tiles are one sweep of 1024 workgroups and 32 tiles that run as quarters; 64 by 4 fill the chip
# once and stay whole; 66 by 1 are quarters only.
@pytest.mark.parametrize("H,I,rows", [(1024, 64, [65] * 32 + [0, 31, 33]), (256, 64, [64] * 60 + [1, 63, 32, 33])])
def test_whole_tiles_and_quarters(H, I, rows):
    _whole_tiles_and_quarters("f32_quarters", H, I, rows)


def _whole_tiles_and_quarters(name, H, I, rows):
    from gpu_common import check_backward, check_forward, run_backward, run_forward, small_config
    cfg = small_config(name, sum(rows), H, I, len(rows), len(rows), 0, 1, "f32", 73)
    inp = make_inputs(cfg, with_dy=True)
    inp["logits"][:] = -10.0
    inp["logits"][np.arange(cfg.T), np.random.default_rng(5).permutation(np.repeat(np.arange(len(rows)), rows))] = 1.0
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k)
    assert ref["counts"].tolist() == rows
    run = run_forward(cfg, inp, store_h1=True)
    check_forward(run, ref, "f32", store_h1=True)
    # the single launch multiplies whole tiles, or strips where a tile has at most 16 rows: the same chain of sums
    single = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True)
    assert torch.equal(single.out, run.out)
    check_backward(run_backward(cfg, inp, run), oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"]), ref["counts"], "f32")
