"""Weight gradients: which kernels take which experts, and both gradients as one launch (one stream) or one launch each (two
streams).  Output shapes that the register-stationary kernel takes for neither, for w1_grad only, for both; experts without
rows, up to and above its 384 rows.  Against the fp64 oracle, and the two forms of launch bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

ROWS = [0, 5, 390, 64, 384, 700]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("rows", [ROWS, [3, 0, 70]], ids=["large_experts", "small_experts"])
@pytest.mark.parametrize("H,I,dtype", [(192, 64, "bf16"), (256, 192, "bf16"), (384, 256, "bf16"), (256, 256, "bf16"), (192, 128, "f32")])
def test_one_launch_or_two(H, I, dtype, rows, keep_xp):
    from gpu_common import check_backward, run_backward, run_forward, small_config
    cfg = small_config("wgrad_launches", sum(rows), H, I, len(rows), len(rows), 0, 1, dtype, 93)
    inp = make_inputs(cfg, with_dy=True)
    inp["logits"][:] = -10.0
    inp["logits"][np.arange(cfg.T), np.random.default_rng(6).permutation(np.repeat(np.arange(len(rows)), rows))] = 1.0
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k)
    run = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
    one = run_backward(cfg, inp, run)
    check_backward(one, oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"]), ref["counts"], dtype)
    two = run_backward(cfg, inp, run, wgrad_stream=torch.cuda.Stream())
    for n in ("dw_gate_up", "dw_down", "dx"):
        assert torch.equal(getattr(one, n), getattr(two, n)), n
