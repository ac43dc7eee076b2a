"""Grouped GEMMs as a weight stream (largest expert of at most 64 rows, 128 where that is a single round): the edges of its
shapes, against the fp64 oracle and bit for bit against the single launch, which runs the same products through the ordinary
tiles (both sum K in the same order).  Where a test means one form of the stream, it asks the rule which one it gets."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23764_amd as moe
import stream_rule
from workloads import make_inputs

pytestmark = pytest.mark.gpu


def _forms(rows, H, I):
    """Forms (tests/stream_rule.py) of GEMM-1, GEMM-2, act_grad and gate_grad on this device; None: tiles."""
    G = -(-torch.cuda.get_device_properties(0).multi_processor_count // 8) * 8
    n_act = sum(r > 0 for r in rows)
    return [stream_rule.form(max(rows), n_act, N, swiglu, G) for N, swiglu in ((I, True), (H, False), (I, False), (H, False))], G


def _shape(form):
    return form and (form.cols, form.rows)


CASES = [
    # name, H, I, rows per expert (repeated over the experts)
    ("one_row", 128, 64, [1, 0, 0]),                        # one expert; 64 columns per item, a single stage
    ("narrow_16", 320, 192, [16, 1, 0, 9]),                 # 16-row stages; K = 2.5 and 1.5 stages of 128
    ("narrow_32", 192, 320, [17, 32, 3]),                   # 32-row stages with 64 columns
    ("wide_32", 448, 832, [32, 2, 31, 0] * 12),             # 256 columns (GEMM-1), 128 (act_grad), 64; N = 3.5 and 6.5 tiles of 128
    ("wide_64", 320, 448, [64, 33, 1, 0, 50]),              # two row blocks
    ("many_rows", 128, 192, [40] * 64),                     # more rows than the token table in LDS holds
    ("above", 192, 128, [65, 3]),                           # above 64 rows, a single round
]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_weight_stream(case, keep_xp):
    _run(*case, keep_xp)


# rows of nine experts, eight of each: 64 experts have rows, 880 and 2072 in all (the token table in LDS holds 2048)
ONE_32, ONE_64 = [32, 3, 17, 1, 0, 9, 26, 2, 20], [64, 50, 1, 33, 0, 7, 52, 18, 34]

DEEP = [
    # name, H, I, rows per expert, columns per item of GEMM-1, GEMM-2, act_grad, gate_grad
    ("gemm1_256_rows_32", 576, 832, ONE_32 * 8, (256, 128, 128, 128)),
    ("gemm1_256_rows_64", 576, 832, ONE_64 * 8, (256, 128, 128, 128)),
    ("gemm1_128_rows_32", 576, 576, ONE_32 * 8, (128, 128, 128, 128)),
    ("gemm1_128_rows_64", 576, 576, ONE_64 * 8, (128, 128, 128, 128)),
    # two stages to an item, fewer than any ring holds: GEMM-1 and act_grad (K = H) ...
    ("short_k_h", 128, 832, ONE_64 * 8, (256, None, 128, None)),
    # ... GEMM-2 (K = I, one stage) and gate_grad (K = 2 I)
    ("short_k_i", 1088, 64, ONE_32 * 8, (None, 128, None, 128)),
]


# GEMM-1: 320 items of 256 columns are one round of 256 workgroups and 64 items that run as 128 of 128 columns
MIXED = [("gemm1_256_then_128_rows_32", 576, 640, ONE_32 * 8), ("gemm1_256_then_128_rows_64", 128, 640, ONE_64 * 8)]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", MIXED, ids=[c[0] for c in MIXED])
def test_whole_rounds_wide_and_the_rest_narrow(case, keep_xp):
    _, H, I, rows = case
    forms, G = _forms(rows, H, I)
    assert _shape(forms[0]) == (256, 32 if max(rows) <= 32 else 64) and forms[0].whole == G and G < forms[0].items < 2 * G
    _run(*case, keep_xp)


# 65..128 rows at the upper edge of a single round of 128-column items, where items of 256 columns (stages of 64 rows) would be
# more than half a round: I / 64 odd; the last: I / 64 even, where they never are
ABOVE_64 = [("i64", 128, 64, 160), ("i320", 128, 320, 48), ("i704_22", 192, 704, 22), ("i704_23", 128, 704, 23), ("i832", 128, 832, 19),
            ("i1600", 192, 1600, 10), ("i1408", 128, 1408, 11)]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("largest", [65, 128])
@pytest.mark.parametrize("case", ABOVE_64, ids=[c[0] for c in ABOVE_64])
def test_rows_above_64_at_the_edge_of_a_round(case, largest, keep_xp):
    name, H, I, n_act = case
    rows = ([largest, 1, 64, 33, largest, 16] * 27)[:n_act]
    assert _shape(_forms(rows, H, I)[0][0]) == (128, 128)
    _run(f"{name}_{largest}", H, I, rows, keep_xp)


MEDIUM = [
    # name, H, I, rows per expert; (columns per item, rows of a stage) of GEMM-1, GEMM-2, act_grad, gate_grad, None: tiles
    # 33..128 rows in a single round: 64 columns per item (stages of 64 and 128 rows, K = 2.5 and 1.5 stages) ...
    ("narrow_64", 320, 192, [64, 33, 1, 0], [(64, 64)] * 4),
    ("narrow_128", 320, 192, [128, 97, 65, 0, 1], [(64, 128)] * 4),
    # ... 128 columns (20 experts with rows: 64 columns would be 440, 260 and 260 items; act_grad 220 of 64) ...
    ("one_round_128", 832, 704, [128, 97, 65, 2, 0] * 5, [(128, 128), (128, 128), (64, 128), (128, 128)]),
    # ... and what takes the tiles: 260 items of 128 columns in GEMM-1, 129 rows
    ("two_rounds", 192, 832, [65, 128] * 10, [None, (64, 128), (128, 128), (64, 128)]),
    ("rows_129", 192, 128, [129, 5], [None] * 4),
]


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", MEDIUM, ids=[c[0] for c in MEDIUM])
def test_single_round_above_32_rows(case, keep_xp):
    name, H, I, rows, want = case
    assert [_shape(f) for f in _forms(rows, H, I)[0]] == want
    _run(name, H, I, rows, keep_xp)


@pytest.mark.parametrize("keep_xp", [True, False])
@pytest.mark.parametrize("case", DEEP, ids=[c[0] for c in DEEP])
def test_several_items_per_workgroup(case, keep_xp):
    """Each workgroup runs more than one item: stages of the next one requested while the last ones of this one are
    multiplied, stores between the loads, and a last round that only some workgroups have an item in."""
    name, H, I, rows, columns = case
    forms, G = _forms(rows, H, I)
    for want, f in zip(columns, forms):
        if want is not None:
            assert f.cols == want and f.whole == f.items > G and f.items % G, (name, f, G)
    _run(name, H, I, rows, keep_xp)


def _run(name, H, I, rows, keep_xp):
    from gpu_common import check_backward, check_forward, check_routing, run_backward, run_forward, small_config
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
