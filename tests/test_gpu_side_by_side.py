"""Small stacks issue the recomputation of a block in the launches of the gradient step of the block above, where the workspace
holds the layout of two streams.  Against the oracle, and bit for bit against the one-slot workspace, where the chains take turns,
on both sides of the rules: rows, widths of the LayerNorm pair, tiles of the products, heads that the attention launch takes.
And the ordering across two streams for stacks beyond those rules."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, takes_two_streams, to_dev

pytestmark = pytest.mark.gpu
KEYS = ("dX1", "dX2", "X1", "X2", "dparams")

# (mode, blocks, width, heads, hidden, tokens, samples, masked)
CASES = [
    ("fp32", 2, 64, 2, 256, 1, 1, False),          # one row, the fewest blocks with anything below
    ("fp32", 5, 72, 3, 200, 33, 5, True),          # ragged widths, three slots' turns
    ("fp32", 3, 200, 5, 520, 64, 16, False),       # 1024 rows: the last that ride
    ("fp32", 3, 384, 6, 1536, 33, 3, False),
    ("bf16", 2, 64, 2, 256, 1, 1, False),
    ("bf16", 1, 128, 2, 512, 77, 3, False),        # nothing below
    ("bf16", 5, 136, 17, 520, 41, 5, True),        # heads of 8: attention apart; erf form of GELU
    ("bf16", 4, 128, 4, 512, 16, 64, False),       # 256 heads of 32 features, 1024 rows
    ("bf16", 3, 640, 8, 2560, 197, 2, True),       # heads of 80
    ("bf16", 3, 768, 12, 3072, 197, 1, False),
    ("bf16", 3, 512, 8, 2048, 250, 4, False),      # weight gradients in 128x128 tiles that two ranges would share; 1000 rows
    ("bf16", 2, 1288, 23, 2576, 20, 3, False),     # rows too wide for the LayerNorm pair
    ("bf16", 2, 2048, 16, 8192, 9, 2, False),      # weights beyond the memory-side cache: in turn
    ("bf16", 2, 1024, 16, 4096, 100, 4, False),    # eight-wavefront tiles
    ("bf16", 3, 256, 4, 1024, 41, 25, False),      # 1025 rows: weight gradients in a launch of their own
    ("bf16", 3, 96, 3, 384, 49, 45, True),         # 2205 rows, attention of a launch per chain
    ("bf16", 2, 64, 1, 256, 60, 140, False),       # 8400 rows: beyond the LayerNorm pair
    ("fp32", 3, 512, 8, 1536, 33, 3, False),       # weight gradients of 640 tiles
    ("fp32", 3, 64, 2, 264, 43, 25, True),         # 1075 rows
    ("fp32", 2, 64, 4, 128, 3, 192, False),        # 768 heads: the last whose attention goes in one launch
    ("fp32", 2, 64, 4, 128, 3, 193, True),         # 772: apart
]


@pytest.mark.parametrize("mode,blocks,width,heads,hidden,tokens,batch,masked", CASES)
def test_side_by_side_or_in_turn(mode, blocks, width, heads, hidden, tokens, batch, masked):
    cfg = dict(n_blocks=blocks, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode=mode)
    print(f"[case] {cfg} masked={masked}", flush=True)
    flat, params_of, x, dy1, dy2 = make_case(cfg, seed=23)
    c = gpu_cfg(cfg)
    params = to_dev(flat, B.param_dtype(c))
    args = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]
    lens = None
    if masked:
        lens = torch.arange(batch, dtype=torch.int32, device="cuda") * 7 % tokens + 1

    def call(schedule, nbytes):
        guard = 4096
        buf = torch.full((nbytes + guard,), 0xFF, dtype=torch.uint8, device="cuda")
        more = dict(workspace=buf[:nbytes], want_inputs=True)
        if schedule == "reprop":
            r = B.rev_stack_backward_reprop_masked(c, params, *args[:2], lens, *args[2:], **more) if masked else \
                B.rev_stack_backward_reprop(c, params, *args, **more)
        else:
            side = torch.cuda.Stream()
            r = B.rev_stack_backward_pareprop_masked(c, params, *args[:2], lens, *args[2:], side, **more) if masked else \
                B.rev_stack_backward_pareprop(c, params, *args, side, **more)
        torch.cuda.synchronize()
        assert bool((buf[nbytes:] == 0xFF).all())
        return r

    full, small = B.rev_stack_workspace_bytes(c), B.rev_stack_workspace_bytes_reprop(c)
    rep = call("reprop", full)
    for other in (call("reprop", small), call("pareprop", full), call("reprop", full)):
        for k in KEYS:
            assert torch.isfinite(rep[k]).all() and torch.equal(rep[k], other[k]), k
    if not masked:
        ref = O.stack_backward_reversible_chunked(x.astype(np.float64), x[:, ::-1].astype(np.float64), params_of, heads, dy1, dy2, chunk=8)
        compare_backward(cfg, rep, ref, TOL[mode], what=str(cfg))


# 8000 rows and 3.3e9 FLOP of a block's forward: beyond every line
@pytest.mark.parametrize("mode", ["bf16", "fp32"])
def test_two_streams_keep_their_order_under_capture_and_with_late_outputs(mode):
    cfg = dict(n_blocks=4, d_model=128, n_heads=2, d_mlp=512, seq_len=50, batch=160, mode=mode)
    assert takes_two_streams(cfg)
    flat, _, x, dy1, dy2 = make_case(cfg, seed=29)
    c = gpu_cfg(cfg)
    params = to_dev(flat, B.param_dtype(c))
    X, dY1, dY2 = to_dev(x), to_dev(dy1), to_dev(dy2)
    Y1, Y2 = B.rev_stack_forward(c, params, X, X)
    ref = {k: v.clone() for k, v in B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2, want_inputs=True).items()}
    ws, sr, cap, late = B.alloc_workspace(c), torch.cuda.Stream(), torch.cuda.Stream(), (torch.zeros_like(Y1), torch.zeros_like(Y2))
    out = {k: torch.zeros_like(v) for k, v in ref.items()}
    big = torch.ones(4096, 4096, device="cuda") / 4096
    torch.cuda.synchronize()
    with torch.cuda.stream(sr):
        for _ in range(10):
            big = big @ big
        late[0].copy_(Y1)
        late[1].copy_(Y2)
    B.rev_stack_backward_pareprop(c, params, *late, dY1, dY2, sr, workspace=ws, want_inputs=True, out=out)
    torch.cuda.synchronize()
    for k in KEYS:
        assert torch.equal(out[k], ref[k]), k
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(cap):
        with torch.cuda.graph(graph, stream=cap):
            B.rev_stack_backward_pareprop(c, params, Y1, Y2, dY1, dY2, sr, workspace=ws, want_inputs=True, out=out)
    torch.cuda.synchronize()
    for rep in range(3):
        for v in out.values():
            v.zero_()
        ws.fill_(0x7F)
        eager = B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(out[k], ref[k]), (rep, k)
        assert torch.equal(eager["dparams"], ref["dparams"])


# Launches of several families are families of their own, and hold what the others lose: the same products under every order
@pytest.mark.parametrize("mode", ["bf16", "fp32"])
def test_timed_families_hold_their_own_work_under_every_order(mode):
    cfg = dict(n_blocks=3, d_model=128, n_heads=2, d_mlp=512, seq_len=50, batch=4, mode=mode)
    flat, _, x, dy1, dy2 = make_case(cfg, seed=41)
    c = gpu_cfg(cfg)
    params = to_dev(flat, B.param_dtype(c))
    args = [to_dev(a) for a in (x, x, dy1, dy2)]

    def families(nbytes):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        B.rev_profile_begin()
        B.rev_stack_backward_reprop(c, params, *args, workspace=ws)
        return B.rev_profile_end()

    turn, side = families(B.rev_stack_workspace_bytes_reprop(c)), families(B.rev_stack_workspace_bytes(c))
    rows, D = cfg["batch"] * cfg["seq_len"], cfg["d_model"]
    products = 2.0 * rows * D * (4 * D + 2 * cfg["d_mlp"])           # of a block's forward; its backward has twice as much
    attention = 4.0 * rows * cfg["seq_len"] * D
    for f in (turn, side):
        assert sum(w for _, _, w, flops in f.values() if flops) == cfg["n_blocks"] * 3 * (products + attention)
    assert [turn[k][1] for k in ("ln_fwd", "ln_bwd", "ln_pair")] == [6, 6, 0]
    assert [side[k][1] for k in ("ln_fwd", "ln_bwd", "ln_pair")] == [3, 3, 3]
    # in turn: the attention forward by itself; side by side only that of the top block, and the attention backward of the bottom one
    # shares its launch with weight gradients (bf16)
    assert turn["attn_fwd"][1:3] == (3, 3 * attention) and side["attn_fwd"][1:3] == (1, attention)
    assert side["attn_bwd"][1:3] == ((0, 0.0) if mode == "bf16" else (1, 2 * attention))
    assert turn["gemm_wgrad"][1] == side["gemm_wgrad"][1] == 0 and side["mixed"][1] == (6 if mode == "bf16" else 5)
