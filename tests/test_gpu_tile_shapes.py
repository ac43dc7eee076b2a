"""Tiles of both shapes one after the other in the same workgroup: rounds of full wide tiles whose last one is halved into tall
items, at reductions of 3 n and 3 n + 1 steps of 64 (the weight stages that the wide tile's last copies go to).  Bit for bit
against the single launch, whose workgroups pass barriers between any two tiles."""
import numpy as np
import pytest
import torch

import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,I", [(2304, 1152), (2368, 1216)])
@pytest.mark.parametrize("keep_xp", [True, False])
def test_halved_round_behind_full_tiles(H, I, keep_xp):
    from gpu_common import run_forward, small_config
    # 9 experts of two tiles: the die with two of them has 2 * 2 * 9 or 2 * 2 * 10 items for its 32 workgroups
    rows = [512 - 13 * i for i in range(9)]
    cfg = small_config("shapes", sum(rows), H, I, 9, 9, 0, 1, "bf16", 91)
    inp = make_inputs(cfg)
    inp["logits"][:] = -10.0
    inp["logits"][np.arange(cfg.T), np.random.default_rng(5).permutation(np.repeat(np.arange(9), rows))] = 1.0
    single = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True, keep_xp=keep_xp)
    assert single.saved.counts.tolist() == rows
    for _ in range(3):
        run = run_forward(cfg, inp, store_h1=True, keep_xp=keep_xp)
        for n in ("A", "H1", "Yp"):
            assert torch.equal(getattr(run.saved, n)[:cfg.T], getattr(single.saved, n)[:cfg.T]), n
        assert torch.equal(run.out, single.out)
