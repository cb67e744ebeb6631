"""The work a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``op`` says which entry points one pass goes through:

* ``backward``  the reversible backward of a stack (``schedule``: ``reprop``, ``pareprop`` or ``static``, the
  allocation-free form of ``reprop``), with or without a key-padding mask, with or without the reconstructed inputs;
* ``forward``   the forward map of a stack (evaluation, or the first half of a training step);
* ``train``     a whole training step: forward, reversible backward, AdamW on all parameters;
* ``merge``     the transition between two stages of a hierarchical model, forward and backward;
* ``adamw`` / ``sgd``  the optimizer update of a packed parameter vector.

All values are synthetic: activations and cotangents standard normal, weight matrices normal with standard deviation
0.02 cut at two of them, LayerNorm gains near 1, small biases.  The two residual streams share their larger part, as
the outputs of a stack that was fed one embedding in both streams do.
"""
import math

import torch

from paper_2306_09342_amd import binding as B
from paper_2306_09342_amd import synth


def _stack(name, op, cfg, **more):
    return dict(name=name, op=op, **dict(cfg, schedule="pareprop", masked=False, want_inputs=False, **more))


def listed():
    c = synth.CONFIGS
    stage1 = synth.HIERARCHIES["swin_t"]["stages"][0]
    return [
        # the smallest stack: a test model or a toy problem in float32; everything is launch latency
        _stack("tiny_fp32", "backward", c["tiny"]),
        # one image: fine-tuning or saliency at batch 1, the inputs wanted back; latency and weight traffic
        dict(_stack("vit_b_batch1", "backward", dict(c["vit_b"], batch=1)), schedule="reprop", want_inputs=True),
        # the benchmark's headline: an image model at its training batch, the two-stream schedule
        _stack("vit_b", "backward", c["vit_b"]),
        # a whole optimisation step of the smaller image model at its training batch
        _stack("vit_s_train", "train", c["vit_s"]),
        # evaluation of the smaller image model on the last, incomplete batch of a data set
        _stack("vit_s_forward_37", "forward", dict(c["vit_s"], batch=37)),
        # text classification: padded sequences of different lengths, the one-stream schedule
        dict(_stack("roberta_base_masked", "backward", c["roberta_base"]), schedule="reprop", masked=True),
        # the largest configured stack: 32 wide blocks
        _stack("vit_h", "backward", c["vit_h"]),
        # the first stage of a window-attention hierarchy: narrow, very many short sequences
        _stack("window_stage1", "backward", stage1),
        # the transition behind that stage, streams fused by averaging
        dict(name="merge_average", op="merge", **synth.merge_cfgs(synth.HIERARCHIES["swin_t"])[0]),
        # the second transition of the widest hierarchy, streams fused by the small MLP
        dict(name="merge_mlp", op="merge", **synth.merge_cfgs(synth.HIERARCHIES["swin_l"], fusion="mlp")[1]),
        # the optimizer on the parameters of the smaller image model, with the bf16 copy the stack reads
        dict(name="adamw_vit_s", op="adamw", n=B.rev_stack_param_count(B.make_cfg(**c["vit_s"])), bf16_copy=True),
        # full precision on a few images: a reference run, or debugging a bf16 one
        dict(_stack("vit_s_fp32", "backward", dict(c["vit_s"], n_blocks=3, batch=3, mode="fp32")), schedule="reprop",
             want_inputs=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_stack(rng, mode, most_flops, most_tokens):
    head_dim = rng.choice((32, 64, 64, 80))
    heads = rng.randint(1 if head_dim > 32 else 2, 1280 // head_dim if mode == "bf16" else 512 // head_dim)
    width = head_dim * heads
    mlp = 4 * width if rng.random() < 0.75 else 8 * rng.randint(width // 4, width // 2)      # ragged hidden widths too
    tokens = _log_int(rng, 16, most_tokens)
    if width % 32 or mlp % 32:
        most_flops = min(most_flops, 1e11)
    cfg = dict(n_blocks=1, d_model=width, n_heads=heads, d_mlp=mlp, seq_len=tokens, batch=1, mode=mode)
    one = 3 * _unit_flops(cfg)                                                                # one block, one sample
    samples = max(1.0, math.exp(rng.uniform(0.0, math.log(max(1.1, most_flops / one)))))
    cfg["n_blocks"] = _log_int(rng, 1, max(1, min(24, int(samples))))
    cfg["batch"] = max(1, min(int(samples / cfg["n_blocks"]), 200000 // tokens, 65535 // heads))
    return cfg


def draw(rng):
    kind = rng.choice(("backward",) * 5 + ("forward", "train", "fp32", "merge", "optimizer"))
    if kind == "merge":
        window = rng.choice((2, 4, 7, 7))
        gh, gw = (2 * window * rng.randint(1, max(1, 28 // window)) for _ in range(2))
        width = 8 * _log_int(rng, 4, 96)
        images = _log_int(rng, 1, max(1, min(128, int(2e8 / (gh * gw * width * 4)))))
        return dict(op="merge", batch=images, grid_h=gh, grid_w=gw, window=window, d_in=width, mode="bf16", ln_eps=1e-5,
                    fusion=rng.choice(("average", "mlp")))
    if kind == "optimizer":
        return dict(op=rng.choice(("adamw", "adamw", "sgd")), n=_log_int(rng, 1000, 100_000_000), bf16_copy=rng.random() < 0.75)
    if kind == "fp32":
        cfg = _draw_stack(rng, "fp32", 4e10, 256)
    else:
        cfg = _draw_stack(rng, "bf16", 1e13, 1024)
    op = kind if kind in ("forward", "train") else "backward"
    schedule = rng.choice(("pareprop", "reprop")) if op != "forward" else "pareprop"
    masked = op != "train" and rng.random() < 0.25
    if op == "backward" and not masked and B.rev_stack_workspace_bytes_reprop(B.make_cfg(**cfg)) <= B.STATIC_WORKSPACE_BYTES \
            and rng.random() < 0.25:
        schedule = "static"
    return dict(op=op, **cfg, schedule=schedule, masked=masked, want_inputs=op == "backward" and rng.random() < 0.25)


# ---- inputs -------------------------------------------------------------------------------------------------------
def _normal(g, *shape):
    return torch.randn(shape, device="cuda", generator=g)


def _streams(g, *shape):
    base = _normal(g, *shape)
    return base + 0.5 * _normal(g, *shape), base + 0.5 * _normal(g, *shape)


def _weights(g, n):
    return _normal(g, n).clamp_(-2.0, 2.0).mul_(0.02)


def _stack_params(g, c):
    flat = _weights(g, B.rev_stack_param_count(c))
    for blk in range(c.n_blocks):
        for t in (0, 6):                                   # the two LayerNorm gains
            off, n = B.rev_stack_param_offset(c, blk, t)
            flat[off:off + n].mul_(5.0).add_(1.0)
    return flat


def _prepare_stack(case, g):
    c = B.make_cfg(**{k: case[k] for k in ("n_blocks", "d_model", "n_heads", "d_mlp", "seq_len", "batch", "mode")})
    shape = (c.batch, c.seq_len, c.d_model)
    flat = _stack_params(g, c)
    s = dict(op=case["op"], schedule=case["schedule"], want_inputs=case["want_inputs"], c=c, side=torch.cuda.Stream(),
             params=flat.to(B.param_dtype(c)), in1=None, in2=None, key_len=None, out={})
    s["in1"], s["in2"] = _streams(g, *shape)              # stack outputs for a backward pass, inputs for a forward pass
    if case["masked"]:
        lens = torch.randint(max(1, c.seq_len // 8), c.seq_len + 1, (c.batch,), device="cuda", generator=g, dtype=torch.int32)
        lens[0] = c.seq_len
        s["key_len"] = lens
    if s["schedule"] != "static":
        s["ws"] = B.alloc_workspace(c, reprop_only=s["schedule"] == "reprop" or s["op"] == "forward")
    if s["op"] != "backward":
        s["Y1"], s["Y2"] = torch.empty(shape, device="cuda"), torch.empty(shape, device="cuda")
    if s["op"] != "forward":
        s["dY1"], s["dY2"] = _normal(g, *shape), _normal(g, *shape)
        if s["key_len"] is not None:                       # nothing flows back into padded positions
            valid = (torch.arange(c.seq_len, device="cuda")[None, :] < s["key_len"][:, None]).unsqueeze(-1)
            s["dY1"].mul_(valid)
            s["dY2"].mul_(valid)
        s["out"] = {k: torch.empty(shape, device="cuda")
                    for k in ("dX1", "dX2") + (("X1", "X2") if s["want_inputs"] else ())}
        s["out"]["dparams"] = torch.empty(flat.numel(), device="cuda")
    if s["op"] == "train":
        s["master"] = s["params"].float() if c.mode == B.REV_MODE_BF16 else s["params"]
        s["m"], s["v"], s["step"] = torch.zeros_like(s["master"]), torch.zeros_like(s["master"]), 0
    return s


def _prepare_merge(case, g):
    c = B.make_merge_cfg(**{k: case[k] for k in ("batch", "grid_h", "grid_w", "window", "d_in", "mode", "ln_eps", "fusion")})
    rows = c.batch * c.grid_h * c.grid_w
    flat = _weights(g, B.rev_merge_param_count(c))
    flat[:4 * c.d_in].mul_(5.0).add_(1.0)                  # the LayerNorm gain
    X1, X2 = _streams(g, rows, c.d_in)
    return dict(op="merge", c=c, params=flat.to(B.param_dtype(c)), X1=X1, X2=X2, dA=_normal(g, rows // 4, 2 * c.d_in),
                dB=_normal(g, rows // 4, 2 * c.d_in), ws=torch.empty(B.rev_merge_workspace_bytes(c), dtype=torch.uint8, device="cuda"),
                merged=torch.empty(rows // 4, 2 * c.d_in, device="cuda"),
                out=dict(dX1=torch.empty_like(X1), dX2=torch.empty_like(X1), dparams=torch.empty(flat.numel(), device="cuda")))


def _prepare_optimizer(case, g):
    n = case["n"]
    s = dict(op=case["op"], master=_weights(g, n), grad=_normal(g, n).mul_(1e-2), step=0,
             copy=torch.empty(n, dtype=torch.bfloat16, device="cuda") if case["bf16_copy"] else None)
    if s["op"] == "adamw":
        s["m"], s["v"] = torch.zeros_like(s["master"]), torch.zeros_like(s["master"])
    return s


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["op"] == "merge":
        return _prepare_merge(case, g)
    if case["op"] in ("adamw", "sgd"):
        return _prepare_optimizer(case, g)
    return _prepare_stack(case, g)


# ---- one pass -------------------------------------------------------------------------------------------------------
def _forward(s):
    c, mask = s["c"], s["key_len"]
    if mask is not None:
        return B.rev_stack_forward_masked(c, s["params"], s["in1"], s["in2"], mask, workspace=s["ws"], Y1=s["Y1"], Y2=s["Y2"])
    return B.rev_stack_forward(c, s["params"], s["in1"], s["in2"], workspace=s["ws"], Y1=s["Y1"], Y2=s["Y2"])


def _backward(s, Y1, Y2):
    c, p, mask = s["c"], s["params"], s["key_len"]
    more = dict(want_inputs=s["want_inputs"], out=s["out"])
    if s["schedule"] == "static":
        return B.rev_stack_backward_reprop_static(c, p, Y1, Y2, s["dY1"], s["dY2"], s["out"])
    if s["schedule"] == "reprop":
        if mask is not None:
            return B.rev_stack_backward_reprop_masked(c, p, Y1, Y2, mask, s["dY1"], s["dY2"], workspace=s["ws"], **more)
        return B.rev_stack_backward_reprop(c, p, Y1, Y2, s["dY1"], s["dY2"], workspace=s["ws"], **more)
    if mask is not None:
        return B.rev_stack_backward_pareprop_masked(c, p, Y1, Y2, mask, s["dY1"], s["dY2"], s["side"], workspace=s["ws"], **more)
    return B.rev_stack_backward_pareprop(c, p, Y1, Y2, s["dY1"], s["dY2"], s["side"], workspace=s["ws"], **more)


def run(state):
    s = state
    if s["op"] == "forward":
        return _forward(s)
    if s["op"] == "backward":
        return _backward(s, s["in1"], s["in2"])
    if s["op"] == "train":
        Y1, Y2 = _forward(s)
        res = _backward(s, Y1, Y2)
        s["step"] += 1
        B.rev_adamw_step(s["master"], res["dparams"], s["m"], s["v"], s["step"], lr=1e-5, params_bf16=s["params"])
        return dict(res, Y1=Y1, Y2=Y2, master=s["master"], params=s["params"], m=s["m"], v=s["v"])
    if s["op"] == "merge":
        merged = B.rev_merge_forward(s["c"], s["params"], s["X1"], s["X2"], workspace=s["ws"], out=s["merged"])
        return dict(B.rev_merge_backward(s["c"], s["params"], s["X1"], s["X2"], s["dA"], s["dB"], workspace=s["ws"],
                                         out=s["out"]), merged=merged)
    if s["op"] == "adamw":
        s["step"] += 1
        B.rev_adamw_step(s["master"], s["grad"], s["m"], s["v"], s["step"], lr=1e-4, params_bf16=s["copy"])
        return dict(master=s["master"], m=s["m"], v=s["v"], copy=s["copy"])
    B.rev_sgd_step(s["master"], s["grad"], 1e-3, params_bf16=s["copy"])
    return dict(master=s["master"], copy=s["copy"])


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _unit_flops(c):
    """One block's forward: the four linear maps and the two attention contractions."""
    tokens, D = c["batch"] * c["seq_len"], c["d_model"]
    return 2.0 * tokens * D * (4 * D + 2 * c["d_mlp"]) + 4.0 * tokens * c["seq_len"] * D


def work(case):
    if case["op"] in ("adamw", "sgd"):
        adam, n = case["op"] == "adamw", float(case["n"])
        return dict(bytes=n * ((28 if adam else 12) + (2 if case["bf16_copy"] else 0)), flops=n * (14 if adam else 2))
    if case["op"] == "merge":
        C, rows = case["d_in"], float(case["batch"] * case["grid_h"] * case["grid_w"])
        mlp = case["fusion"] == "mlp"
        params = 8 * C + 8 * C * C + (3 * C * C + 2 * C if mlp else 0)
        es = 2 if case["mode"] == "bf16" else 4
        flops = 2.0 * (rows / 4) * 2 * C * 4 * C + (2.0 * rows * 3 * C * C if mlp else 0.0)
        return dict(bytes=rows * C * 4 * (4 + 1.5) + params * (es + 4.0), flops=3 * flops)
    act = 4.0 * case["batch"] * case["seq_len"] * case["d_model"]
    D, Dm = case["d_model"], case["d_mlp"]
    params = float(case["n_blocks"]) * (4 * D * D + 2 * D * Dm + 9 * D + Dm)
    es = 2 if case["mode"] == "bf16" else 4
    unit = case["n_blocks"] * _unit_flops(case)
    if case["op"] == "forward":
        return dict(bytes=params * es + 4 * act, flops=unit)
    bytes_, flops = params * (es + 4) + (8 if case["want_inputs"] else 6) * act, 3 * unit
    if case["op"] == "train":                              # Y1, Y2 written and read; the optimizer reads the gradient again
        bytes_ += 4 * act + params * (28 + (2 if case["mode"] == "bf16" else 0))
        flops += unit + 14 * params
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    if case["op"] in ("adamw", "sgd"):
        return dict(rel=1e-5, max=8e-3 if case["bf16_copy"] else 1e-4)     # one step of the last place of the bf16 copy
    return dict(rel=1e-2) if case["mode"] == "bf16" else dict(rel=2e-5)
