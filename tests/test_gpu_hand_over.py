"""Hand-over between tasks of the bf16 single launches in both forms: behind one die's L2 (few tasks per worker) and through memory,
with workers that draw from other dies' queues once their own has run out (more than four tasks per worker; skewed rows, so that the
queues end at different times).  Which form a launch takes follows from its number of tasks, counted here from its queues: forwards with
and without a permuted copy and backwards in either form.  The serialized launches give the same bits."""
import numpy as np
import pytest
import torch

import paper_2605_23764_amd as moe
from plan_check import decode_plan
from workloads import make_inputs

pytestmark = pytest.mark.gpu


def hands_far(shape, workspace, backward):
    lay = moe.moe_ffn_debug_layout(shape, backward=backward)
    tasks = sum(len(q) for q in decode_plan(workspace.cpu().numpy(), lay).queues)
    workers = (torch.cuda.get_device_properties(0).multi_processor_count + 7) // 8 * 8
    print("  backward" if backward else "  forward", tasks, "tasks,", workers, "workers", flush=True)
    return tasks > 4 * workers


# fwd_far, bwd_far: the form that the launches of 256 workers take
@pytest.mark.parametrize("T,H,I,skew,keep_xp,fwd_far,bwd_far", [
    (12000, 128, 192, True, True, True, False), (12000, 128, 192, True, False, False, False), (9000, 1024, 128, False, True, True, False),
    (9000, 1024, 128, True, False, False, False), (700, 192, 128, True, True, False, False),
    (12000, 1024, 704, True, False, True, True), (12000, 1024, 704, False, True, True, True)])
def test_single_launch_equals_serialized(T, H, I, skew, keep_xp, fwd_far, bwd_far):
    from gpu_common import run_backward, run_forward, small_config
    cfg = small_config(f"hand_over_{T}_{H}", T, H, I, 16, 16, 0, 4, "bf16", 98)
    inp = make_inputs(cfg, with_dy=True)
    if skew:
        inp["logits"] = inp["logits"] - 0.35 * np.arange(16, dtype=np.float32)[None, :]
    ser = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
    want = run_backward(cfg, inp, ser)
    R = int(ser.saved.offsets.cpu()[-1])
    for again in range(3):
        print(cfg.name, "skew", skew, "Xp", keep_xp, "pass", again, flush=True)
        per = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True, keep_xp=keep_xp)
        assert moe.moe_ffn_last_status(per.shape, per.workspace) == 0
        for name in ("Xp", "H1", "A", "Yp"):
            if getattr(per.saved, name) is not None:
                assert torch.equal(getattr(ser.saved, name)[:R], getattr(per.saved, name)[:R]), name
        assert torch.equal(ser.out, per.out)
        assert hands_far(per.shape, per.workspace, False) == fwd_far
        got = run_backward(cfg, inp, per, mode=moe.MODE_PERSISTENT)
        assert hands_far(per.shape, got.workspace, True) == bwd_far
        for name in ("dx", "dw_gate_up", "dw_down", "dtopk_w"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name
