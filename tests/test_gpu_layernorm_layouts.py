"""LayerNorm layouts: rows of up to 256 floats share a wavefront in long inputs, short inputs take the block of eight rows.  All add
a row in one order, so the bits of a sample must not depend on the number of rows; the gradients of all rows together
(gains, biases: the column sums) must match the oracle."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, to_dev

pytestmark = pytest.mark.gpu

# (width, heads, tokens, samples, fewer samples): every layout of narrow rows on both sides of 16384 rows (forward) and 8192
# (backward); one row, 7, 8 and 9 rows; the widest row of the short kernel and one beyond; accumulators in LDS; rows of 1024 on
# both sides of 2048 rows, of 96 beyond 100000
CASES = [(32, 1, 7, 2400, 3), (64, 2, 7, 2400, 3), (96, 3, 7, 2400, 1), (128, 4, 7, 2400, 3), (160, 2, 7, 2400, 3), (256, 4, 7, 2400, 3),
         (264, 11, 7, 1171, 3), (800, 10, 7, 1171, 1), (1280, 16, 9, 1, 1), (1288, 23, 8, 1, 1), (64, 2, 1, 1, 1), (200, 5, 7, 1, 1),
         (1024, 16, 7, 300, 3), (96, 3, 7, 14300, 3)]


@pytest.mark.parametrize("mode", ["bf16", "fp32"])
@pytest.mark.parametrize("width,heads,tokens,batch,few", CASES)
def test_rows_have_the_same_bits_in_every_layout(width, heads, tokens, batch, few, mode):
    cfg = dict(n_blocks=1, d_model=width, n_heads=heads, d_mlp=32, seq_len=tokens, batch=batch, mode=mode)
    print(f"[case] {cfg}", flush=True)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=7)
    dev = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]

    def run(b):
        c = gpu_cfg(dict(cfg, batch=b))
        params = to_dev(flat, B.param_dtype(c))
        X1, X2, dY1, dY2 = (a[:b].contiguous() for a in dev)
        Y1, Y2 = B.rev_stack_forward(c, params, X1, X2)
        res = B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2, want_inputs=True)
        torch.cuda.synchronize()
        return Y1, Y2, res

    Y1, Y2, res = run(batch)
    if few < batch:
        y1, y2, r = run(few)
        assert torch.equal(y1, Y1[:few]) and torch.equal(y2, Y2[:few])
        for k in ("dX1", "dX2", "X1", "X2"):
            assert torch.equal(r[k], res[k][:few]), k
    ref = O.stack_backward_reversible_chunked(Y1.cpu().numpy(), Y2.cpu().numpy(), blocks, heads, dy1, dy2, chunk=256)
    compare_backward(cfg, res, ref, TOL[mode], what=str(cfg))
