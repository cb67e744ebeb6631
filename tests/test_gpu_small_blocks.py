"""Small blocks on one stream: QKV's input gradient, the weight gradients, the column sums and the second stages of sums in one
launch, on both sides of the rules that choose it, against the oracle, in both workspaces; the schedule of two streams, which
issues them apart, must give the same bits, also where the calls on one stream issue them together.  Three blocks, so that sums of one
block are finished by the launch of the next."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, takes_two_streams, to_dev

pytestmark = pytest.mark.gpu

# (mode, width, heads, hidden, tokens, samples)
CASES = [
    ("fp32", 72, 3, 200, 1, 1),            # one row
    ("fp32", 136, 17, 520, 32, 32),         # 1024 rows, the last whose column sums come in one piece; ragged widths
    ("fp32", 136, 17, 520, 41, 25),         # 1025 rows
    ("fp32", 384, 6, 1536, 33, 3),         # weight gradients of 432 64x64 tiles, together still
    ("fp32", 512, 8, 1536, 33, 3),         # 640: apart
    ("fp32", 384, 6, 1536, 64, 16),        # together on one stream, apart on two
    ("bf16", 72, 3, 200, 1, 1),            # 32x32 tiles
    ("bf16", 136, 17, 520, 41, 25),        # 1025 rows: two ranges of tokens
    ("bf16", 264, 11, 1032, 32, 32),       # 1024 rows, 64x64 tiles
    ("bf16", 768, 12, 3072, 197, 1),       # 32x32 tiles, the rest fills the chip
    ("bf16", 768, 12, 3072, 197, 4),       # together on one stream, apart on two
    ("bf16", 1024, 16, 4096, 197, 4),      # larger tiles: apart
]


def test_each_type_has_a_case_with_one_order_of_the_chains_per_schedule():
    orders = {}
    for mode, width, heads, hidden, tokens, batch in CASES:
        c = gpu_cfg(dict(n_blocks=3, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode=mode))
        full, small = B.rev_stack_workspace_bytes(c), B.rev_stack_workspace_bytes_reprop(c)
        orders.setdefault(mode, set()).add((B.rev_stack_backward_order(c, False, full), B.rev_stack_backward_order(c, True, full)))
        assert B.rev_stack_backward_order(c, False, small) == B.REV_ORDER_IN_TURN
    for mode in ("fp32", "bf16"):
        assert (B.REV_ORDER_SIDE_BY_SIDE, B.REV_ORDER_TWO_STREAMS) in orders[mode], orders


@pytest.mark.parametrize("mode,width,heads,hidden,tokens,batch", CASES)
def test_one_launch_or_several(mode, width, heads, hidden, tokens, batch):
    cfg = dict(n_blocks=3, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode=mode)
    print(f"[case] {cfg} two streams: {takes_two_streams(cfg)}", flush=True)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=19)
    c = gpu_cfg(cfg)
    params = to_dev(flat, B.param_dtype(c))
    args = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]
    rep = B.rev_stack_backward_reprop(c, params, *args, want_inputs=True)
    small = torch.empty(B.rev_stack_workspace_bytes_reprop(c), dtype=torch.uint8, device="cuda")
    again = B.rev_stack_backward_reprop(c, params, *args, workspace=small, want_inputs=True)
    par = B.rev_stack_backward_pareprop(c, params, *args, torch.cuda.Stream(), want_inputs=True)
    torch.cuda.synchronize()
    for k in ("dX1", "dX2", "X1", "X2", "dparams"):
        assert torch.equal(rep[k], par[k]) and torch.equal(rep[k], again[k]), k
    ref = O.stack_backward_reversible_chunked(x.astype(np.float64), x[:, ::-1].astype(np.float64), blocks, heads, dy1, dy2, chunk=8)
    compare_backward(cfg, rep, ref, TOL[mode], what=str(cfg))


# 1000 rows of 512: weight gradients that a launch of their own would sum in two ranges, in one piece for any number of blocks
@pytest.mark.parametrize("mode,width,heads,hidden,tokens,batch", [
    ("bf16", 512, 8, 2048, 250, 4), ("bf16", 768, 12, 3072, 197, 1), ("bf16", 136, 17, 520, 41, 25), ("fp32", 136, 17, 520, 32, 32)])
def test_a_block_has_the_same_gradients_in_a_stack_of_any_depth(mode, width, heads, hidden, tokens, batch):
    cfg = dict(n_blocks=3, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode=mode)
    print(f"[case] {cfg}", flush=True)
    flat, _, x, dy1, dy2 = make_case(cfg, seed=37)
    deep, one = gpu_cfg(cfg), gpu_cfg(dict(cfg, n_blocks=1))
    params = to_dev(flat, B.param_dtype(deep))
    per = B.rev_stack_param_count(one)
    args = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]
    top = params[-per:].clone()
    ref = B.rev_stack_backward_reprop(deep, params, *args)["dparams"][-per:]
    rep = B.rev_stack_backward_reprop(one, top, *args)["dparams"]
    par = B.rev_stack_backward_pareprop(one, top, *args, torch.cuda.Stream())["dparams"]
    torch.cuda.synchronize()
    assert torch.equal(rep, ref) and torch.equal(par, ref)
