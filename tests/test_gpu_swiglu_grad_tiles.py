"""SwiGLU_grad epilogue of the act_grad tiles, whose pre-activations come through LDS block by block: tiles whose last block is
partial, whose wave rows hold different numbers of blocks, with the register-fed block, tall, and with half a column block."""
import numpy as np
import pytest

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# rows per expert: one tile of every shape, and wave rows of 0 to 4 blocks; the largest is above 128, so the launch runs as tiles
COUNTS = [[129, 1, 31, 33, 64, 65, 0, 97], [257, 288, 289, 320, 256, 225, 191, 2], [321, 384, 350, 0, 700, 641, 160, 5]]


@pytest.mark.parametrize("I", [64, 192, 320])
@pytest.mark.parametrize("counts", COUNTS, ids=["one_wave_row", "register_fed", "tall_and_split"])
def test_act_grad_tiles(counts, I):
    from gpu_common import check_backward, run_backward, run_forward, small_config
    cfg = small_config(f"grad_tiles_{I}", sum(counts), 192, I, 8, 8, 0, 1, "bf16", 97)
    inp = make_inputs(cfg, with_dy=True)
    owner = np.repeat(np.arange(8), counts)
    np.random.default_rng(6).shuffle(owner)
    logits = np.full((cfg.T, 8), -4.0, dtype=np.float32)
    logits[np.arange(cfg.T), owner] = 4.0
    inp["logits"] = logits
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k, cfg.expert_base, cfg.E_local)
    assert ref["counts"].tolist() == counts
    ref_b = oracle.backward(inp["dy"], ref, inp["w_gate_up"], inp["w_down"])
    run = run_forward(cfg, inp, store_h1=True)
    for mode in (moe.MODE_SERIALIZED, moe.MODE_PERSISTENT):
        print(cfg.name, counts, "mode", mode, flush=True)
        check_backward(run_backward(cfg, inp, run, mode=mode), ref_b, ref["counts"], cfg.dtype)
