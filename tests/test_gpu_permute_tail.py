"""Dispatch of rows whose last pass is full for some lanes of a wave only (a row is 16-byte vectors, 4, 7 or 14 to a lane and pass), with odd
numbers of rows per wave: single launches and the one launch per operator copy each row once, and nothing behind the last row."""
import numpy as np
import pytest
import torch

import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu


# vectors per row: 840 and 888 (a remainder of 392..447 of 7 * 64), 1744 (848..895 of 14 * 64), 208 (192..255 of 4 * 64); 848, 1760, 240
@pytest.mark.parametrize("dtype,H", [("bf16", 6720), ("bf16", 7104), ("bf16", 13952), ("bf16", 1664), ("f32", 3392), ("f32", 7040), ("f32", 960)])
@pytest.mark.parametrize("T", [65, 301])
def test_rows_are_copied_once(dtype, H, T):
    from gpu_common import run_forward, small_config
    cfg = small_config(f"permute_tail_{H}", T, H, 64, 7, 7, 0, 3, dtype, 95)
    inp = make_inputs(cfg)
    inp["logits"] = inp["logits"] - 0.2 * np.arange(7, dtype=np.float32)[None, :]
    print(cfg.name, dtype, "T", T, flush=True)
    ser = run_forward(cfg, inp, store_h1=True)
    R = 3 * T
    x = ser.dev["x"]
    args = (ser.shape, x, ser.dev["logits"], ser.dev["w_gate_up"], ser.dev["w_down"])
    calls = [(moe.moe_ffn_forward, moe.MODE_SERIALIZED), (moe.moe_ffn_forward, moe.MODE_PERSISTENT)]
    if dtype == "bf16":
        calls += [(moe.moe_ffn_forward_scatter, moe.MODE_SERIALIZED), (moe.moe_ffn_forward_scatter, moe.MODE_PERSISTENT)]
    for forward, mode in calls:
        for again in range(2):
            saved = moe.alloc_saved(ser.shape, store_h1=True)
            padded = torch.full((R + 16, H), 7.0, dtype=x.dtype, device="cuda")    # every row is local: Xp ends with the last one
            saved.Xp = padded[:R]
            out = torch.full_like(ser.out, float("nan"))
            forward(*args, out, saved, ser.workspace, mode)
            torch.cuda.synchronize()
            assert moe.moe_ffn_last_status(ser.shape, ser.workspace) == 0
            assert int(saved.offsets[-1]) == R
            assert torch.equal(saved.Xp, x[saved.token_of[:R].long()]), (forward.__name__, mode)
            assert bool((padded[R:] == 7.0).all()), (forward.__name__, mode)
            assert torch.equal(saved.H1[:R], ser.saved.H1[:R]), (forward.__name__, mode)
            if forward is moe.moe_ffn_forward:
                assert torch.equal(out, ser.out), mode
