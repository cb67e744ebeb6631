"""256x256 and 256x128 tiles of the bf16 GEMMs: row and column counts that the last tiles overhang (they are moved back and store
only their own part), against the oracle, and sample bits against launches that take small tiles."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, to_dev

pytestmark = pytest.mark.gpu

# (width, heads, hidden, tokens, samples): 2561 rows (one beyond ten tiles) and 5128 columns (eight beyond twenty); 4334 rows;
# 2560 rows and 3840 columns, all tiles whole.  256x128 tiles (fc1 and its transpose): contractions of one, two and three
# stages, 65807, 33005 and 42007 rows, 520, 1024 and 776 columns (QKV too in the last, 576 columns, and
# on two streams its residual and plain products, 192 columns); 256x128 tiles on one stream and
# 256x256 ones on two, whose column sums have the same bits: 12796 rows, 3064 columns
CASES = [(1280, 16, 5128, 197, 13), (768, 12, 3072, 197, 22), (1280, 20, 3840, 64, 40),
         (64, 2, 520, 7, 9401), (192, 6, 776, 7, 6001), (128, 2, 1024, 5, 6601), (640, 10, 3064, 7, 1828)]


@pytest.mark.parametrize("width,heads,hidden,tokens,batch", CASES)
def test_overhanging_tiles_match_the_oracle_and_small_tiles(width, heads, hidden, tokens, batch):
    cfg = dict(n_blocks=1, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode="bf16")
    print(f"[case] {cfg}", flush=True)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=13)
    dev = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]

    def run(b):
        c = gpu_cfg(dict(cfg, batch=b))
        params = to_dev(flat, B.param_dtype(c))
        X1, X2, dY1, dY2 = (a[:b].contiguous() for a in dev)
        Y1, Y2 = B.rev_stack_forward(c, params, X1, X2)
        rep = B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2, want_inputs=True)
        par = B.rev_stack_backward_pareprop(c, params, Y1, Y2, dY1, dY2, torch.cuda.Stream(), want_inputs=True)
        torch.cuda.synchronize()
        for k in ("dX1", "dX2", "X1", "X2", "dparams"):
            assert torch.equal(rep[k], par[k]), k
        return Y1, Y2, rep

    Y1, Y2, res = run(batch)
    y1, y2, few = run(1)
    assert torch.equal(y1, Y1[:1]) and torch.equal(y2, Y2[:1])
    for k in ("dX1", "dX2", "X1", "X2"):
        assert torch.equal(few[k], res[k][:1]), k
    ref = O.stack_backward_reversible_chunked(Y1.cpu().numpy(), Y2.cpu().numpy(), blocks, heads, dy1, dy2, chunk=4 if tokens > 50 else 256)
    compare_backward(cfg, res, ref, TOL["bf16"], what=str(cfg))
