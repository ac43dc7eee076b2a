"""Timed cases of the Dispatch-to-Combine MoE-FFN layer: one GPU's expert-parallel share, through the public entry points.

What a program does with this layer, and the case that stands for it:
  decode     a serving step with few tokens (inference: no activations kept); weight streaming and launch latency
  prefill    a serving step with many tokens, plain or skewed routing, either launch mode or the scatter epilogue
  forward    the training forward: routing results and activations are kept for the backward
  backward   the backward on activations that a forward has left
  train      forward + backward of one layer, the gradients included
each in bf16 or fp32 storage, with and without a permuted copy of the tokens, on one or two streams.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_23764_amd as moe
from workloads import MoeConfig, expert_bias

# One GPU's share of a layer: hidden size, expert width, experts, local experts, first local expert, experts per token.
MID = dict(H=2048, I=1408, E=16, E_local=16, base=0, k=4)         # mid-size layer, every expert local
LARGE = dict(H=7168, I=2048, E=256, E_local=32, base=0, k=8)      # 256 experts over eight GPUs
TINY = dict(H=256, I=128, E=8, E_local=8, base=0, k=2)


def _case(name, kind, T, layer, dtype="bf16", skew=False, mode="serialized", copy=True, scatter=False, two_streams=False):
    return dict(name=name, kind=kind, T=T, **layer, dtype=dtype, skew=skew, mode=mode, copy=copy, scatter=scatter,
                two_streams=two_streams)


def listed():
    return [
        # one token of one sequence: the smallest call there is
        _case("decode_1_mid", "decode", 1, MID),
        # a small serving batch; about 20 of the 32 local experts get one or two rows each
        _case("decode_32_large", "decode", 32, LARGE),
        # a full serving batch: every local expert has a few rows
        _case("decode_256_large", "decode", 256, LARGE),
        # a prompt of ordinary, odd length through the scatter epilogue as a single launch
        _case("prefill_1000_mid_scatter", "prefill", 1000, MID, mode="persistent", scatter=True),
        # many prompt tokens with skewed routing: empty experts beside one with eleven times the mean
        _case("prefill_8192_large_skewed", "prefill", 8192, LARGE, skew=True, mode="persistent"),
        # training forward, matrix bound
        _case("forward_4096_mid", "forward", 4096, MID),
        # training forward at the headline shape
        _case("forward_8192_large", "forward", 8192, LARGE),
        # backward, about a thousand rows per expert, in its fastest form
        _case("backward_4096_mid", "backward", 4096, MID, mode="persistent", two_streams=True),
        # the whole training step at the headline shape: the largest case
        _case("train_8192_large", "train", 8192, LARGE),
        # a training step of odd sizes: width not a multiple of a tile, experts from the middle, no permuted copy
        _case("train_777_odd", "train", 777, dict(H=1088, I=704, E=24, E_local=10, base=6, k=3), copy=False),
        # fp32 storage: the small exact layer, and one of ordinary size
        _case("train_256_tiny_f32", "train", 256, TINY, dtype="f32"),
        _case("train_1500_f32", "train", 1500, dict(H=1024, I=704, E=16, E_local=16, base=0, k=4), dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _any_layer(rng, h_max, i_max):
    E = rng.choice([8, 16, 24, 64, 128, 256])
    E_local = rng.choice([e for e in (4, 8, 10, 16, 32, E) if e <= min(E, 64)])
    return dict(H=64 * _log_int(rng, 4, h_max // 64), I=64 * _log_int(rng, 2, i_max // 64), E=E, E_local=E_local,
                base=rng.randint(0, E - E_local), k=rng.randint(1, min(8, E)))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "forward", "backward", "train", "train"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    bf16 = dtype == "bf16"
    if kind == "decode":
        layer = rng.choice([MID, LARGE, _any_layer(rng, 7168, 2048)]) if bf16 else _any_layer(rng, 2048, 1408)
        T = _log_int(rng, 1, 256)
    else:
        layer = rng.choice([MID, LARGE, _any_layer(rng, 7168, 2048)]) if bf16 else _any_layer(rng, 1024, 704)
        T = _log_int(rng, 256, 8192) if bf16 else _log_int(rng, 64, 1500)
    # not above the largest listed case
    rows = T * layer["k"] * layer["E_local"] / layer["E"]
    while rows * layer["H"] * layer["I"] > 0.9 * 8192 * 7168 * 2048 and T > 64:
        T, rows = T // 2, rows / 2
    mode = rng.choice(["serialized", "serialized", "persistent"])
    if not bf16 and kind in ("backward", "train"):
        mode = "serialized"
    return dict(kind=kind, T=T, **layer, dtype=dtype, skew=rng.random() < 0.25, mode=mode, copy=rng.random() < 0.6,
                scatter=bf16 and kind in ("decode", "prefill") and rng.random() < 0.2,
                two_streams=kind in ("backward", "train") and rng.random() < 0.3)


def _keeps(case):
    return case["kind"] in ("forward", "backward", "train")


def _inputs(case, seed):
    T, H, I, E, El = (case[n] for n in ("T", "H", "I", "E", "E_local"))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def normal(shape, dtype, scale=1.0):
        t = torch.randn(shape, generator=g, device="cuda", dtype=dtype)
        return t.mul_(scale) if scale != 1.0 else t

    inp = dict(x=normal((T, H), dt), logits=normal((T, E), torch.float32),
               w_gate_up=normal((El, H, 2 * I), dt, H ** -0.5), w_down=normal((El, I, H), dt, I ** -0.5))
    if case["skew"]:
        inp["logits"] += _bias(case).cuda()[None, :]
    if case["kind"] in ("backward", "train"):
        inp["dy"] = normal((T, H), dt)
    return inp


def _bias(case):
    """Zipf-like bias per expert; the ranks are the same for every seed, so that the load keeps its shape."""
    return torch.from_numpy(expert_bias(MoeConfig("skew", case["T"], case["H"], case["I"], case["E"], case["E_local"],
                                                  case["base"], case["k"], case["dtype"], 1004, True)))


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    dt = s["x"].dtype
    s["shape"] = shape = moe.make_shape(case["T"], case["H"], case["I"], case["E"], case["E_local"], case["base"], case["k"], dt)
    s["mode"] = moe.MODE_PERSISTENT if case["mode"] == "persistent" else moe.MODE_SERIALIZED
    s["ws"] = moe.alloc_workspace(shape)
    s["out"] = torch.empty_like(s["x"])
    s["saved"] = None
    if _keeps(case):
        s["saved"] = moe.alloc_saved(shape, store_h1=True, keep_xp=case["copy"])
        for n in ("Xp", "H1", "A", "Yp"):      # rows past the last one in use are never written
            if getattr(s["saved"], n) is not None:
                getattr(s["saved"], n).zero_()
    if case["kind"] in ("backward", "train"):
        s["ws_b"] = moe.alloc_workspace(shape, backward=True)
        s["dx"], s["dw_gate_up"], s["dw_down"] = (torch.empty_like(s[n]) for n in ("x", "w_gate_up", "w_down"))
        s["dtopk_w"] = torch.empty(case["T"], case["k"], dtype=torch.float32, device="cuda")
        s["side"] = torch.cuda.Stream() if case["two_streams"] else None
    if case["kind"] == "backward":
        _forward(s, moe.MODE_SERIALIZED)
    return s


def _forward(s, mode):
    call = moe.moe_ffn_forward_scatter if s["case"]["scatter"] else moe.moe_ffn_forward
    call(s["shape"], s["x"], s["logits"], s["w_gate_up"], s["w_down"], s["out"], s["saved"], s["ws"], mode)


def _backward(s):
    args = (s["shape"], s["dy"], s["x"], s["w_gate_up"], s["w_down"], s["saved"], s["dx"], s["dw_gate_up"], s["dw_down"],
            s["dtopk_w"], s["ws_b"])
    if s["side"] is not None:
        moe.moe_ffn_backward_two_streams(*args, s["side"], s["mode"])
    else:
        moe.moe_ffn_backward(*args, s["mode"])


def run(s):
    kind, sv = s["case"]["kind"], s["saved"]
    got = {}
    if kind != "backward":
        _forward(s, s["mode"])
        got["out"] = s["out"]
    if _keeps(s["case"]) and kind != "backward":
        got.update(topk_idx=sv.topk_idx, topk_w=sv.topk_w, counts=sv.counts, row_of=sv.row_of, A=sv.A, H1=sv.H1, Yp=sv.Yp)
    if kind in ("backward", "train"):
        _backward(s)
        got.update(dx=s["dx"], dw_gate_up=s["dw_gate_up"], dw_down=s["dw_down"], dtopk_w=s["dtopk_w"])
    return got


def _load(case):
    """Expected (rows, experts with rows, tokens with a local expert) of the routing."""
    T, E, El, base, k = (case[n] for n in ("T", "E", "E_local", "base", "k"))
    if not case["skew"]:
        rows, p = T * k * El / E, k / E
        tokens = T * (1.0 - math.prod((E - El - i) / (E - i) if E - El > i else 0.0 for i in range(k)))
        return rows, El * (1.0 - (1.0 - p) ** T), tokens
    g = np.random.Generator(np.random.PCG64(1))
    n = min(T, 2048)
    lg = g.standard_normal((n, E), dtype=np.float32) + _bias(case).numpy()[None, :]
    top = np.argpartition(-lg, k - 1, axis=1)[:, :k] - base
    here = (top >= 0) & (top < El)
    share = np.bincount(top[here], minlength=El) / n
    return here.sum() * T / n, float((1.0 - (1.0 - share) ** T).sum()), float(here.any(axis=1).mean() * T)


def work(case):
    T, H, I, E, El, k = (case[n] for n in ("T", "H", "I", "E", "E_local", "k"))
    eb = 2 if case["dtype"] == "bf16" else 4
    rows, active, tokens = _load(case)
    weights = active * 3 * H * I * eb
    nbytes = flops = 0.0
    if case["kind"] != "backward":
        nbytes += T * E * 4 + tokens * H * eb + weights + T * H * eb
        flops += 6.0 * rows * H * I
        if _keeps(case):
            nbytes += T * k * 12 + rows * (3 * I + H + (H if case["copy"] else 0)) * eb
    if case["kind"] in ("backward", "train"):
        nbytes += tokens * H * eb + T * H * eb + T * k * 12          # dY in, dX and the routing weights' gradient out
        if case["kind"] == "backward":                              # a training step has the activations and weights read above
            nbytes += rows * (3 * I + 2 * H) * eb + weights
        nbytes += El * 3 * H * I * eb
        flops += 12.0 * rows * H * I
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times the distance from the 64-bit result: up to 1.1e-6 in fp32; up to 3.8e-3 in bf16, which stores every
    # intermediate rounded (the scatter epilogue also rounds every partial sum).
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1.5e-2, "max": 0.15}


def exact(case, seed):
    """The layer in 64 bits, expert by expert, nothing rounded in between."""
    T, H, I, El, base, k = (case[n] for n in ("T", "H", "I", "E_local", "base", "k"))
    inp = _inputs(case, seed)
    f64 = dict(dtype=torch.float64, device="cuda")
    lg = inp["logits"].double()
    order = torch.argsort(lg, dim=1, descending=True, stable=True)[:, :k]
    w = torch.softmax(torch.gather(lg, 1, order), dim=1)
    local = order - base
    here = (local >= 0) & (local < El)
    x = inp["x"].double()
    r_max = T * min(k, El)
    out = torch.zeros(T, H, **f64)
    keep, grads = _keeps(case), case["kind"] in ("backward", "train")
    if keep:
        sv = dict(A=torch.zeros(r_max, I, **f64), H1=torch.zeros(r_max, 2 * I, **f64), Yp=torch.zeros(r_max, H, **f64))
        row_of = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
        counts = torch.zeros(El, dtype=torch.int32, device="cuda")
    if grads:
        dy = inp["dy"].double()
        dx = torch.zeros(T, H, **f64)
        dw1 = torch.zeros(El, H, 2 * I, **f64)
        dw2 = torch.zeros(El, I, H, **f64)
        dtw = torch.zeros(T, k, **f64)
    r0 = 0
    for e in range(El):
        t, j = torch.nonzero(here & (local == e), as_tuple=True)     # ascending token
        n = t.numel()
        if keep:
            counts[e] = n
            row_of[t, j] = torch.arange(r0, r0 + n, dtype=torch.int32, device="cuda")
        if n == 0:
            continue
        w1, w2 = inp["w_gate_up"][e].double(), inp["w_down"][e].double()
        xe = x[t]
        h = xe @ w1
        g, u = h[:, :I], h[:, I:]
        sg = torch.sigmoid(g)
        a = g * sg * u
        y = a @ w2
        we = w[t, j][:, None]
        out.index_add_(0, t, we * y)
        if keep:
            sv["A"][r0:r0 + n], sv["H1"][r0:r0 + n], sv["Yp"][r0:r0 + n] = a, h, y
        if grads:
            dye = dy[t]
            dtw[t, j] = (dye * y).sum(1)
            dyp = we * dye
            da = dyp @ w2.t()
            dw2[e] = a.t() @ dyp
            dh = torch.cat([da * u * sg * (1.0 + g * (1.0 - sg)), da * g * sg], 1)
            dw1[e] = xe.t() @ dh
            dx.index_add_(0, t, dh @ w1.t())
        r0 += n
    got = {}
    if case["kind"] != "backward":
        got["out"] = out
    if keep and case["kind"] != "backward":
        got.update(topk_idx=order.to(torch.int32), topk_w=w, counts=counts, row_of=row_of, **sv)
    if grads:
        got.update(dx=dx, dw_gate_up=dw1, dw_down=dw2, dtopk_w=dtw)
    return got
