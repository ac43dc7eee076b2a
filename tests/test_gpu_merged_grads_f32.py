"""fp32 backward of small layers on one stream: gate_grad and both weight gradients as one launch.  The two-stream call runs the same
tiles as launches of their own: same bits, and the oracle."""
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# rows and widths around a tile of 64 and its quarters, more and fewer tiles than workgroups, experts without rows, no local row
CASES = [(1, 64, 64, 2, 2, 0, 1), (1, 64, 64, 8, 1, 7, 1), (65, 128, 64, 4, 4, 0, 1), (256, 256, 128, 8, 8, 0, 2), (300, 512, 448, 16, 10, 3, 4),
         (40, 1024, 704, 64, 32, 0, 6), (700, 192, 320, 5, 5, 0, 5)]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", CASES, ids=["T%d_H%d_I%d_E%d_%d_%d_k%d" % c for c in CASES])
def test_one_launch_equals_three(case, keep_xp):
    from gpu_common import check_backward, run_backward, run_forward, small_config
    cfg = small_config("merged_T%d" % case[0], *case, "f32", 83)
    inp = make_inputs(cfg, with_dy=True)
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k, cfg.expert_base, cfg.E_local)
    ref_b = oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"])
    run = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
    print(cfg.name, case, "Xp", keep_xp, flush=True)
    one = run_backward(cfg, inp, run)
    two = run_backward(cfg, inp, run, wgrad_stream=torch.cuda.Stream())
    for name in ("dx", "dw_gate_up", "dw_down", "dtopk_w"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    check_backward(one, ref_b, ref["counts"], cfg.dtype)
