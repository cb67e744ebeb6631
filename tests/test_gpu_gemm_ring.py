"""64x128, 128x128 and 192x128 tiles of the bf16 GEMMs' deep ring: one row beyond whole tiles, columns and contractions that
end inside a tile and a stage, the fused column sums of each strip height, against the oracle; PaReprop must equal Reprop, and a
sample alone (in the smallest tiles) the same sample in the batch, bit for bit."""
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, to_dev

pytestmark = pytest.mark.gpu

# (width, heads, hidden, tokens, samples).  2607 rows, contractions of 648 and 1304 (a last chunk of 8, of 24): 64x128, and 128x128 for fc1
# and its transpose; 1900 rows, 1288 wide: 128x128 for all but QKV; 6305 rows, 760 wide: 192x128; 3204 rows: 192x128 with column
# sums, 1160 wide, 1544 hidden; 2560 rows, 880 wide: weight gradients in 256x128 tiles, whose column sums are held to the chunks that
# 128x128 tiles would have; 201 and 335 rows, 1160 wide: on both sides of the line up to which 64x64 tiles stand in for 64x128; 1067 rows, 960
# wide, and 2051 rows, 640 wide: on both sides of the line up to which more than 160 eight-wavefront tiles give way on two streams
CASES = [(648, 9, 1304, 79, 33), (1288, 23, 1288, 95, 20), (760, 19, 2056, 65, 97), (1160, 29, 1544, 89, 36), (880, 11, 2480, 32, 80),
         (1160, 29, 4648, 67, 3), (1160, 29, 4648, 67, 5), (960, 12, 3840, 97, 11), (640, 8, 2560, 293, 7)]


@pytest.mark.parametrize("width,heads,hidden,tokens,batch", CASES)
def test_ring_tiles_match_the_oracle_and_small_tiles(width, heads, hidden, tokens, batch):
    cfg = dict(n_blocks=1, d_model=width, n_heads=heads, d_mlp=hidden, seq_len=tokens, batch=batch, mode="bf16")
    print(f"[case] {cfg}", flush=True)
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=17)
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
    ref = O.stack_backward_reversible_chunked(Y1.cpu().numpy(), Y2.cpu().numpy(), blocks, heads, dy1, dy2, chunk=8)
    compare_backward(cfg, res, ref, TOL["bf16"], what=str(cfg))
