"""Ranks of more tokens than workgroups of one sub-chunk (32 tokens) fit on the chip: a workgroup then takes several in a row.  Integers
are exact; the launch with Dispatch in it and the one without, both around the first size with two sub-chunks to a workgroup (the last
workgroup with one or two, the last sub-chunk ragged), and where the sub-chunks per workgroup do not divide their number."""
import numpy as np
import pytest
import torch

import paper_2605_23764_amd as moe
from oracle.moe_ffn_oracle import local_permutation, route
from workloads import MoeConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over,E,E_local,base,k", [(0, 16, 16, 0, 4), (1, 16, 16, 0, 4), (33, 70, 65, 3, 5), (32 * 1024 + 31, 24, 10, 6, 3),
                                                    (3 * 32 * 1024 + 1, 8, 1, 7, 2)])
def test_ranks_of_many_tokens(over, E, E_local, base, k):
    from gpu_common import check_routing, run_forward
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T = 4 * cus * 32 + over
    cfg = MoeConfig("rank_subs", T, 64, 64, E, E_local, base, k, "bf16", 92)
    print("T", T, "E_local", E_local, flush=True)
    rng = np.random.default_rng(over)
    inp = dict(x=torch.from_numpy(rng.standard_normal((T, 64), dtype=np.float32)).bfloat16().float().numpy(),
               logits=rng.standard_normal((T, E), dtype=np.float32) - 0.05 * np.arange(E, dtype=np.float32)[None, :],
               w_gate_up=np.zeros((E_local, 64, 128), np.float32), w_down=np.zeros((E_local, 64, 64), np.float32))
    ref = dict(zip(("topk_idx", "topk_w"), route(inp["logits"], k)))
    ref.update(zip(("counts", "offsets", "row_of", "token_of", "slot_of"), local_permutation(ref["topk_idx"], base, E_local)))
    run = run_forward(cfg, inp)                       # Dispatch in the launch
    check_routing(run, ref)
    R = int(ref["offsets"][-1])
    assert torch.equal(run.saved.Xp[:R], run.dev["x"][torch.from_numpy(ref["token_of"]).long().cuda()])
    run = run_forward(cfg, inp, keep_xp=False)        # ranks alone
    check_routing(run, ref)
    run = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT)
    assert moe.moe_ffn_last_status(run.shape, run.workspace) == 0
    check_routing(run, ref)
