"""GEMMs at the edges of every tile of the dispatch, through whole blocks against the
float64 oracle (bf16): K shorter than one stage, a short last stage in each kernel, stages whose second half is empty,
ragged rows and columns, the fused column sums of each strip height; the float32 products: both tile sizes,
a token count that is no multiple of anything, heads of every width class with masks.  PaReprop must equal Reprop bit for bit."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, oracle_forward, rel_err, to_dev

pytestmark = pytest.mark.gpu

SHAPES = {
    # 32x32 and 64x64 tiles
    "one_token_K8": dict(n_blocks=1, d_model=8, n_heads=1, d_mlp=8, seq_len=1, batch=1),
    "ragged_K40": dict(n_blocks=2, d_model=40, n_heads=1, d_mlp=72, seq_len=33, batch=1),
    "tiles64_K328": dict(n_blocks=1, d_model=328, n_heads=1 + 40, d_mlp=2248, seq_len=197, batch=1),
    # 32x32 tiles at K = 256 / 264 (the last of three stages holds one chunk of 8) and 2048, 64x64 tiles at the same short K
    "groups3_K256": dict(n_blocks=1, d_model=256, n_heads=4, d_mlp=2048, seq_len=75, batch=8),
    "groups3_K264": dict(n_blocks=1, d_model=264, n_heads=3, d_mlp=2056, seq_len=75, batch=8),
    # 128x128 tiles at K = 144, 64x64 at 2056
    "groups2_K144": dict(n_blocks=1, d_model=144, n_heads=2, d_mlp=2056, seq_len=150, batch=10),
    # 64x128 tiles in the ring (fc2 and its transpose; a last chunk of 8) and in two stages (proj, fc1, its transpose with column sums)
    "ring64x128_K1544": dict(n_blocks=1, d_model=384, n_heads=6, d_mlp=1544, seq_len=197, batch=23),
    "two_stage64x128_K1288": dict(n_blocks=1, d_model=1288, n_heads=23, d_mlp=1288, seq_len=95, batch=20),
    # few output columns at many rows
    "whole_K72": dict(n_blocks=1, d_model=72, n_heads=1, d_mlp=200, seq_len=31, batch=100),
    "whole_rows3073": dict(n_blocks=1, d_model=64, n_heads=1, d_mlp=136, seq_len=439, batch=7),
    # weight gradients in 256x256 tiles: one token beyond the last full stage; ragged in every direction; three token ranges,
    # the last one short
    "wgrad256_one_token_over": dict(n_blocks=1, d_model=1024, n_heads=16, d_mlp=4096, seq_len=683, batch=3),
    "wgrad256_ragged": dict(n_blocks=1, d_model=776, n_heads=97, d_mlp=3080, seq_len=125, batch=20),
    "wgrad256_ranges": dict(n_blocks=1, d_model=520, n_heads=13, d_mlp=2056, seq_len=353, batch=17),
}


F32_SHAPES = {
    "f32_wide_output": dict(n_blocks=1, d_model=72, n_heads=3, d_mlp=1544, seq_len=67, batch=21),
    "f32_wide_wgrad": dict(n_blocks=1, d_model=512, n_heads=16, d_mlp=2048, seq_len=37, batch=1),
    "f32_heads104": dict(n_blocks=1, d_model=208, n_heads=2, d_mlp=16, seq_len=161, batch=2),
    "f32_heads72": dict(n_blocks=2, d_model=72, n_heads=1, d_mlp=40, seq_len=129, batch=2),
}


@pytest.mark.parametrize("name,mode", [(n, "bf16") for n in SHAPES] + [(n, "fp32") for n in F32_SHAPES] + [("f32_heads104", "bf16")])
def test_gemm_shapes_match_the_oracle(name, mode):
    cfg = dict(SHAPES.get(name) or F32_SHAPES[name], mode=mode)
    tol = TOL[mode]
    print(f"[case] {name} {cfg}", flush=True)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=3)
    x2 = x[:, ::-1].copy()
    y1, y2 = oracle_forward(cfg, blocks, x, x2)
    y1f, y2f = y1.astype(np.float32), y2.astype(np.float32)
    ref = O.stack_backward_reversible_chunked(y1f, y2f, blocks, cfg["n_heads"], dy1, dy2)
    c = gpu_cfg(cfg)
    params = to_dev(flat, B.param_dtype(c))
    gy1, gy2 = B.rev_stack_forward(c, params, to_dev(x), to_dev(x2))
    args = [to_dev(a) for a in (y1f, y2f, dy1, dy2)]
    rep = B.rev_stack_backward_reprop(c, params, *args, want_inputs=True)
    par = B.rev_stack_backward_pareprop(c, params, *args, torch.cuda.Stream(), want_inputs=True)
    torch.cuda.synchronize()
    assert rel_err(gy1.cpu().numpy(), y1) <= tol and rel_err(gy2.cpu().numpy(), y2) <= tol
    compare_backward(cfg, rep, ref, tol, what=name)
    for k in ("dX1", "dX2", "dparams", "X1", "X2"):
        assert torch.equal(rep[k], par[k]), f"PaReprop differs from Reprop in {k}"


@pytest.mark.parametrize("mode", ["fp32", "bf16"])
def test_masked_wide_heads_match_the_oracle(mode):
    cfg = dict(n_blocks=1, d_model=224, n_heads=2, d_mlp=64, seq_len=100, batch=3, mode=mode)
    lens = np.asarray([100, 1, 65], dtype=np.int32)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=4)
    ref = [O.stack_backward_reversible(x[b:b + 1].astype(np.float64), x[b:b + 1, ::-1].astype(np.float64), blocks, 2,
                                       dy1[b:b + 1].astype(np.float64), dy2[b:b + 1].astype(np.float64), key_len=lens[b:b + 1])
           for b in range(3)]
    c = gpu_cfg(cfg)
    args = [to_dev(a) for a in (x, x[:, ::-1].copy())]
    res = B.rev_stack_backward_reprop_masked(c, to_dev(flat, B.param_dtype(c)), *args, torch.from_numpy(lens).cuda(), to_dev(dy1),
                                             to_dev(dy2))
    torch.cuda.synchronize()
    for i, k in enumerate(("dX1", "dX2")):
        assert rel_err(res[k].cpu().numpy(), np.concatenate([r[i] for r in ref])) <= TOL[mode], k


@pytest.mark.parametrize("tokens,batch", [(3, 1), (100, 64), (100, 200)])
def test_an_infinite_weight_stays_infinite_in_a_contraction_that_ends_inside_a_stage(tokens, batch):
    """What a short last stage reads beyond the contraction counts as zeros, not as 0 times the weights it re-reads: with one
    infinite weight at the last index, Y2 is infinite in its column and finite elsewhere.  32x32, 64x64 and 128x128 tiles."""
    D = 72
    c = B.make_cfg(n_blocks=1, d_model=D, n_heads=1, d_mlp=D, seq_len=tokens, batch=batch, mode="bf16")
    params = torch.zeros(B.rev_stack_param_count(c), device="cuda", dtype=torch.bfloat16)
    b_fc1, n = B.rev_stack_param_offset(c, 0, 9)
    params[b_fc1:b_fc1 + n] = 1.0                                   # the activation is gelu(1) everywhere
    w_fc2, _ = B.rev_stack_param_offset(c, 0, 10)
    params[w_fc2 + 5 * D + D - 1] = float("inf")
    X = torch.ones(batch, tokens, D, device="cuda")
    _, Y2 = B.rev_stack_forward(c, params, X, X)
    torch.cuda.synchronize()
    want = torch.ones(D, device="cuda")
    want[5] = float("inf")
    assert bool((Y2 == want).all())
