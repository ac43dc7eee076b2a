"""Dispatch to Combine of up to 64 tokens as one launch of weight streams: against the launches of the serialized mode bit for bit, and
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# T, H, I, E, E_local, base, k: one token; no local row; items of 64, 128 and 256 columns with whole and mixed rounds; stages of 16, 32
# and 64 rows; columns that do not fill an item; many experts; K of one, two and many stages
CASES = [(1, 64, 64, 2, 2, 0, 1), (1, 2048, 1408, 16, 16, 0, 4), (2, 128, 64, 64, 2, 62, 1), (7, 192, 320, 8, 8, 0, 8),
         (16, 704, 192, 16, 16, 0, 2), (33, 1088, 704, 24, 10, 6, 3), (40, 3200, 2112, 32, 32, 0, 6), (64, 256, 128, 256, 256, 0, 8),
         (64, 4096, 832, 3, 3, 0, 2), (64, 320, 1600, 5, 1, 2, 4), (64, 64, 64, 1, 1, 0, 1)]


def _config(case, seed):
    from gpu_common import small_config
    return small_config("layer_T%d_H%d_I%d" % case[:3], *case, "bf16", seed)


def _launches(run):
    """The serialized launches on the routing of `run`, into fresh buffers."""
    sv = moe.alloc_saved(run.shape, store_h1=True)
    ws = moe.alloc_workspace(run.shape)
    out = torch.full_like(run.out, float("nan"))
    moe.moe_route(run.shape, run.dev["logits"], sv, ws)
    moe.moe_dispatch_to_combine(run.shape, run.dev["x"], run.dev["w_gate_up"], run.dev["w_down"], out, sv, ws, moe.MODE_SERIALIZED)
    return sv, out


def _same(run, sv, out):
    R = int(sv.offsets.cpu()[-1])
    for name in ("topk_idx", "topk_w", "counts", "offsets", "row_of"):
        assert torch.equal(getattr(run.saved, name), getattr(sv, name)), name
    for name in ("token_of", "slot_of", "Xp", "H1", "A", "Yp"):
        if getattr(run.saved, name) is not None:
            assert torch.equal(getattr(run.saved, name)[:R], getattr(sv, name)[:R]), name
    assert torch.equal(run.out, out)


@pytest.mark.parametrize("case", CASES, ids=["T%d_H%d_I%d_E%d_%d_%d_k%d" % c for c in CASES])
@pytest.mark.parametrize("keep_xp", [True, False])
def test_up_to_64_tokens(case, keep_xp):
    from gpu_common import check_forward, check_routing, run_forward
    cfg = _config(case, 71)
    inp = make_inputs(cfg)
    ref = oracle.forward(inp["x"], inp["logits"], inp["w_gate_up"], inp["w_down"], cfg.k, cfg.expert_base, cfg.E_local)
    print(cfg.name, "Xp", keep_xp, flush=True)
    run = run_forward(cfg, inp, mode=moe.MODE_PERSISTENT, store_h1=True, keep_xp=keep_xp)
    assert moe.moe_ffn_last_status(run.shape, run.workspace) == 0
    _same(run, *_launches(run))
    check_routing(run, ref)
    if int(ref["offsets"][-1]):
        check_forward(run, ref, cfg.dtype, store_h1=True)
    else:
        assert not run.out.any()
    # inference, again on the same workspace, other tokens
    run.dev["x"] = torch.roll(run.dev["x"], 1, 1)
    for _ in range(3):
        run.out.fill_(float("nan"))
        moe.moe_ffn_forward(run.shape, run.dev["x"], run.dev["logits"], run.dev["w_gate_up"], run.dev["w_down"], run.out, None, run.workspace,
                            moe.MODE_PERSISTENT)
    assert torch.equal(run.out, _launches(run)[1])


@pytest.mark.parametrize("case", [CASES[1], CASES[2], CASES[5], CASES[7]], ids=["T%d_H%d_I%d" % CASES[i][:3] for i in (1, 2, 5, 7)])
def test_scatter_call_runs_the_same_streams(case):
    """The single launch of the scatter call: out of moe_ffn_forward bit for bit, the caller's Yp untouched."""
    from gpu_common import run_forward
    cfg = _config(case, 77)
    run = run_forward(cfg, make_inputs(cfg))
    args = (run.shape, run.dev["x"], run.dev["logits"], run.dev["w_gate_up"], run.dev["w_down"])
    for saved in (moe.alloc_saved(run.shape, store_h1=True), None):
        out = torch.full_like(run.out, float("nan"))
        if saved is not None:
            saved.Yp.fill_(3.0)
        moe.moe_ffn_forward_scatter(*args, out, saved, run.workspace, moe.MODE_PERSISTENT)
        assert torch.equal(out, run.out)
        assert saved is None or bool((saved.Yp == 3.0).all())
        assert moe.moe_ffn_last_status(run.shape, run.workspace) == 0


def test_second_launch_on_the_same_routing_does_nothing():
    from gpu_common import run_forward
    cfg = _config((33, 1088, 704, 24, 10, 6, 3), 76)
    run = run_forward(cfg, make_inputs(cfg))
    args = (run.shape, run.dev["x"], run.dev["w_gate_up"], run.dev["w_down"])
    moe.moe_route(run.shape, run.dev["logits"], run.saved, run.workspace)
    out, again = torch.empty_like(run.out), torch.full_like(run.out, 7.0)
    moe.moe_dispatch_to_combine(*args, out, run.saved, run.workspace, moe.MODE_PERSISTENT)
    moe.moe_dispatch_to_combine(*args, again, run.saved, run.workspace, moe.MODE_PERSISTENT)
    assert torch.equal(out, run.out) and bool((again == 7.0).all())
    assert moe.moe_ffn_last_status(run.shape, run.workspace) == 0


def test_expired_wait_is_reported_and_the_next_call_is_right():
    """Without polls a wait that is not met at once expires: the launch ends, the status says so, out is as it was (GEMM-1 leaves 80 of 256
    workgroups without a share, whose waits for the others' expire; no token is combined then), and the next call on the workspace is right."""
    from gpu_common import run_forward
    cfg = _config((64, 2048, 704, 16, 16, 0, 4), 73)
    run = run_forward(cfg, make_inputs(cfg), mode=moe.MODE_PERSISTENT)
    args = (run.shape, run.dev["x"], run.dev["logits"], run.dev["w_gate_up"], run.dev["w_down"])
    out = torch.full_like(run.out, 7.0)
    try:
        moe.moe_ffn_debug_set_spin_limit(0)
        for forward in (moe.moe_ffn_forward, moe.moe_ffn_forward_scatter):
            forward(*args, out, run.saved, run.workspace, moe.MODE_PERSISTENT)
            torch.cuda.synchronize()
            assert moe.moe_ffn_last_status(run.shape, run.workspace) == -5
            assert bool((out == 7.0).all()), forward.__name__
    finally:
        moe.moe_ffn_debug_set_spin_limit(1 << 20)
    moe.moe_ffn_forward(*args, out, run.saved, run.workspace, moe.MODE_PERSISTENT)
    torch.cuda.synchronize()
    assert moe.moe_ffn_last_status(run.shape, run.workspace) == 0
    assert torch.equal(out, run.out)


def test_two_streams_side_by_side():
    """Two layers of one token each on two streams, whose launches share the chip in any split."""
    from gpu_common import run_forward
    runs = []
    for seed in (74, 75):
        cfg = _config((1 + seed % 2, 2048, 1408, 16, 16, 0, 4), seed)
        runs.append(run_forward(cfg, make_inputs(cfg), mode=moe.MODE_PERSISTENT))
    want = [r.out.clone() for r in runs]
    streams = [torch.cuda.Stream() for _ in runs]
    torch.cuda.synchronize()
    for i in range(200):
        for r, s in zip(runs, streams):
            with torch.cuda.stream(s):
                moe.moe_ffn_forward(r.shape, r.dev["x"], r.dev["logits"], r.dev["w_gate_up"], r.dev["w_down"], r.out, r.saved, r.workspace,
                                    moe.MODE_PERSISTENT)
    torch.cuda.synchronize()
    for r, w in zip(runs, want):
        assert moe.moe_ffn_last_status(r.shape, r.workspace) == 0
        assert torch.equal(r.out, w)
