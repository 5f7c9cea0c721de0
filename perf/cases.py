"""The layer's work as a user's program has it done: forward-only calls (serving), training steps (forward + backward)
and the stand-alone steps that a caller strings together itself, all through paper_2502_16927_amd.binding.

Letters: T tokens, d model width, r low (dispatch) width, N experts, k experts per token, h expert hidden width.
Shapes are those of paper_2502_16927_amd.synth, a few of them with token counts that divide into nothing.
"""
from __future__ import annotations

import math

import torch

from paper_2502_16927_amd import binding as B

DEV = "cuda:0"
W_STD = 0.02


def _case(name, kind, T, d, r, N, k, h, dtype="bf16", order="dcca", zipf=0.0, capacity=0.0, aux=0.0,
          out_bf16=False, wire_bf16=False, accumulate=False):
    case = dict(kind=kind, T=T, d=d, r=r, N=N, k=k, h=h, dtype=dtype, order=order, zipf=zipf, capacity=capacity, aux=aux,
                out_bf16=out_bf16, wire_bf16=wire_bf16, accumulate=accumulate)
    return dict(case, name=name) if name else case


def listed():
    return [
        # fp32 storage, the debugging and reference precision: a call so small that launches are most of it
        _case("tiny_f32", "infer", 256, 256, 64, 8, 2, 256, dtype="f32"),
        # a decode step of a large layer: few tokens, every expert's weights read
        _case("decode_32", "infer", 32, 4096, 1024, 64, 8, 4096),
        # a decode step of a busy server, y wanted in bf16; the token count is whatever is in flight
        _case("decode_500", "infer", 500, 4096, 1024, 64, 8, 4096, out_bf16=True),
        # a prefill chunk of the same layer
        _case("prefill_2048", "infer", 2048, 4096, 1024, 64, 8, 4096),
        # evaluation of a mid-size layer: forward only on a training-size batch
        _case("medium_infer", "infer", 8192, 1024, 256, 64, 8, 1024),
        # the training step of the same layer
        _case("medium_train", "train", 8192, 1024, 256, 64, 8, 1024),
        # ... with the paper's balancing options (expert capacity 1.2, load-balance loss 0.001) on a ragged batch
        _case("medium_train_balanced", "train", 6001, 1024, 256, 64, 8, 1024, capacity=1.2, aux=0.001),
        # ... and as the fine-grained layer that the paper compares with
        _case("medium_train_cdac", "train", 8192, 1024, 256, 64, 8, 1024, order="cdac"),
        # a large layer inside a gradient-accumulation loop
        _case("xl_train_accumulate", "train", 16384, 2048, 512, 64, 6, 2048, accumulate=True),
        # widths that are no powers of two, a ragged batch, everything that may be bf16 in bf16
        _case("2p7b_train_bf16", "train", 3001, 2560, 640, 64, 8, 2560, out_bf16=True, wire_bf16=True),
        # the largest: 128 experts under skewed routing (rows per expert from a few dozen to about 30 thousand)
        _case("zipf_train", "train", 32768, 4096, 1024, 128, 8, 2048, zipf=1.2),
        # the steps called one by one, as a program does that puts its own exchange between them
        _case("steps_3001", "steps", 3001, 1024, 256, 64, 8, 1024),
    ]


# Work of the largest listed case, which bounds the drawn ones: rows x expert matrix, and expert weights.
_MAX_ROWS_X_MATRIX = 32768 * 8 * 1024 * 2048
_MAX_WEIGHTS = 128 * 1024 * 2048


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["infer", "train", "steps", "f32"], [0.38, 0.40, 0.12, 0.10])[0]
    if kind == "f32":
        d = rng.choice([256, 512])
        return _case(None, "infer", _log_int(rng, 32, 1024), d, d // 4, rng.choice([8, 16]), rng.randint(1, 4), rng.choice([d // 2, d]), dtype="f32")
    while True:
        d = 256 * _log_int(rng, 2, 16)          # 512 .. 4096, r = d / 4
        r = d // 4
        h = rng.choice([d, d, d // 2])
        N = rng.choice([8, 16, 32, 48, 64, 64, 96, 128])
        k = rng.choice([1, 2, 4, 6, 8, 8])
        T = _log_int(rng, 16, 32768) if kind == "infer" else _log_int(rng, 1024, 32768)
        if kind == "steps":
            T = min(T, 8192)
        passes = 3 if kind == "train" else 1
        if T * k * r * h * passes <= 3 * _MAX_ROWS_X_MATRIX and N * r * h <= _MAX_WEIGHTS:
            break
    opts = dict(zipf=rng.choice([0.0, 0.0, 0.0, 0.6, 1.2]), out_bf16=rng.random() < 0.3, wire_bf16=rng.random() < 0.2)
    if kind == "steps":
        return _case(None, kind, T, d, r, N, k, h, zipf=opts["zipf"])
    if rng.random() < 0.15 and d <= 2048:       # the fine-grained order has no bf16 result
        opts.update(order="cdac", out_bf16=False)
    if kind == "train":
        opts["accumulate"] = rng.random() < 0.3
        if rng.random() < 0.2:
            opts.update(capacity=1.2, aux=0.001)
    return _case(None, kind, T, d, r, N, k, h, **opts)


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    T, d, r, N, k, h = (case[n] for n in ("T", "d", "r", "N", "k", "h"))
    f32 = case["dtype"] == "f32"
    dtype = torch.float32 if f32 else torch.bfloat16
    cdac = case["order"] == "cdac"
    win, hid = (d, r) if cdac else (r, h)

    def normal(shape, std, dt=dtype):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, std, generator=g).to(dt)

    flags = (B.FLAG_OUT_BF16 if case["out_bf16"] else 0) | (B.FLAG_WIRE_BF16 if case["wire_bf16"] else 0) | (B.FLAG_ACCUMULATE if case["accumulate"] else 0)
    capacity = B.expert_capacity(T, k, N, case["capacity"]) if case["capacity"] else 0
    dims = B.make_dims(T, d, r, N, k, h, B.F32 if f32 else B.BF16, B.ORDER_CDAC if cdac else B.ORDER_DCCA, flags, capacity=capacity, aux_alpha=case["aux"])
    s = {"kind": case["kind"], "dims": dims, "aux": case["aux"] > 0.0}
    s["x"] = normal((T, d), W_STD if f32 else 1.0)
    s["w_gate"] = normal((d, N), W_STD, torch.float32)
    s["gate_bias"] = None
    if case["zipf"]:
        s["gate_bias"] = -case["zipf"] * torch.log1p(torch.randperm(N, generator=g, device=DEV).float())
    s["w1"], s["w2"] = normal((N, win, hid), W_STD), normal((N, hid, win), W_STD)

    if case["kind"] == "steps":
        s["x_low"] = normal((T, win), 1.0)
        s["idx"] = torch.empty((T, k), dtype=torch.int32, device=DEV)
        s["weights"] = torch.empty((T, k), dtype=torch.float32, device=DEV)
        s["offsets"] = torch.empty(N + 1, dtype=torch.int32, device=DEV)
        s["slot_of"], s["src_of"] = (torch.empty(T * k, dtype=torch.int32, device=DEV) for _ in range(2))
        s["x_perm"], s["o_perm"] = (torch.empty((T * k, win), dtype=dtype, device=DEV) for _ in range(2))
        s["y_low"] = torch.empty((T, win), dtype=torch.float32, device=DEV)
        s["ws_route"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_ROUTE), DEV)
        s["ws_dispatch"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_DISPATCH), DEV)
        s["ws_ffn"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_GROUPED_FFN), DEV)
        return s

    s["w_down"], s["w_up"] = (None, None) if cdac else (normal((d, r), W_STD), normal((r, d), W_STD))
    s["params"] = B.make_params(s["w_down"], s["w_up"], s["w_gate"], s["gate_bias"], s["w1"], s["w2"])
    out_dtype = torch.bfloat16 if case["out_bf16"] else torch.float32
    s["y"] = torch.empty((T, d), dtype=out_dtype, device=DEV)
    if case["kind"] == "infer":
        s["ws"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_LAYER_FORWARD), DEV)
        return s
    s["dy"] = normal((T, d), 1.0)
    s["dx"] = torch.empty((T, d), dtype=out_dtype, device=DEV)
    fresh = torch.zeros if case["accumulate"] else torch.empty    # an accumulation loop starts from zeroed gradients
    s["d_w_down"], s["d_w_up"] = (None, None) if cdac else (fresh((d, r), device=DEV), fresh((r, d), device=DEV))
    s["d_w_gate"], s["d_w1"], s["d_w2"] = fresh((d, N), device=DEV), fresh((N, win, hid), device=DEV), fresh((N, hid, win), device=DEV)
    s["saved"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_SAVED), DEV)
    s["ws"] = B.alloc_bytes(B.workspace_bytes(dims, B.WS_LAYER_TRAIN), DEV)
    if s["aux"]:
        at = B.saved_aux_layout(dims)["aux_loss"]
        s["loss"] = s["saved"][at:at + 4].view(torch.float32)
    return s


def run(s):
    dims = s["dims"]
    if s["kind"] == "steps":
        B.bigmac_route(dims, s["x"], s["w_gate"], s["gate_bias"], s["idx"], s["weights"], None, s["ws_route"])
        B.bigmac_dispatch(dims, s["x_low"], s["idx"], s["x_perm"], s["offsets"], s["slot_of"], s["src_of"], s["ws_dispatch"])
        B.bigmac_grouped_ffn(dims, s["x_perm"], s["offsets"], s["w1"], s["w2"], None, s["o_perm"], s["ws_ffn"])
        B.bigmac_combine(dims, s["o_perm"], s["slot_of"], s["weights"], s["y_low"])
        return {n: s[n] for n in ("idx", "weights", "offsets", "slot_of", "src_of", "x_perm", "o_perm", "y_low")}
    if s["kind"] == "infer":
        B.bigmac_layer_forward(dims, s["params"], s["x"], s["y"], None, s["ws"])
        return s["y"]
    B.bigmac_layer_forward(dims, s["params"], s["x"], s["y"], s["saved"], s["ws"])
    B.bigmac_layer_backward(dims, s["params"], s["x"], s["dy"], s["saved"], s["dx"], s["d_w_down"], s["d_w_up"], s["d_w_gate"],
                            s["d_w1"], s["d_w2"], s["ws"])
    return {n: s[n] for n in ("y", "dx", "d_w_down", "d_w_up", "d_w_gate", "d_w1", "d_w2") + (("loss",) if s["aux"] else ())}


def work(case):
    T, d, r, N, k, h = (case[n] for n in ("T", "d", "r", "N", "k", "h"))
    es = 4 if case["dtype"] == "f32" else 2
    out = 2 if case["out_bf16"] else 4
    cdac = case["order"] == "cdac"
    win, hid = (d, r) if cdac else (r, h)
    reached = N * (1.0 - (1.0 - k / N) ** T)                      # experts with at least one token, evenly popular
    expert_matrices = 2.0 * reached * win * hid
    shared = 0.0 if cdac else 2.0 * d * r
    router = 2.0 * T * d * N
    experts = 4.0 * T * k * win * hid
    if case["kind"] == "steps":
        rows = T * k
        moved = T * d * es + d * N * 4 + T * win * es + expert_matrices * es + 2 * rows * win * es + T * win * 4 + 16 * rows
        return {"bytes": moved, "flops": router + experts + 2.0 * rows * win}
    flops = router + experts + (0.0 if cdac else 4.0 * T * d * r)
    moved = T * d * es + d * N * 4 + (expert_matrices + shared) * es + T * d * out
    if case["kind"] == "infer":
        return {"bytes": moved, "flops": flops}
    gradients = (2.0 * N * win * hid + shared + d * N) * 4 * (2 if case["accumulate"] else 1)
    return {"bytes": moved + T * d * es + T * d * out + gradients, "flops": 3.0 * flops}


def tolerance(case):
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
