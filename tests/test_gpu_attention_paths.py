"""bf16 attention of heads with 32, 64 or 80 features: which kernel a launch takes (both backward passes in one launch with
workgroups of two or of four wavefronts, one workgroup per head, one launch per pass) follows from the batch, so the bits of
a sample must not depend on it, and the samples must match the oracle.  Token counts lie at the edges of the 32-row
wavefronts, the 64-row tiles and the ring of two tiles."""
import numpy as np
import pytest
import torch

from oracle import rev_oracle as O
from paper_2306_09342_amd import binding as B

from parity_util import TOL, compare_backward, gpu_cfg, make_case, rel_err, to_dev

pytestmark = pytest.mark.gpu

# (features, tokens, batches, masked); two heads.  A launch of both passes has 4 * batch * ceil(tokens / 128) workgroups of four
# wavefronts; it is taken up to 768 of them, 512 where one workgroup per head is the other choice for 64 features.
CASES = [
    (80, 1, (2, 60, 200), False),
    (80, 33, (3, 60, 200), True),
    (80, 64, (2, 200), False),
    (80, 129, (2, 40, 100), True),
    (80, 257, (2, 20, 70), False),
    (64, 32, (2, 60, 140), False),
    (64, 65, (3, 40, 140), True),
    (64, 193, (2, 20, 70), False),
    (64, 300, (2, 20, 70), True),
    (32, 31, (2, 60, 200), False),
    (32, 97, (3, 60, 200), True),
    (32, 257, (2, 70), True),
    # forward tiles of 32 rows: up to 8 tokens, and up to 16 where heads * tokens <= 131072
    (32, 8, (2, 60), True),
    (64, 16, (2, 4200), True),
    (80, 13, (3, 5100), False),
]


@pytest.mark.parametrize("dh,tokens,batches,masked", CASES)
def test_every_path_gives_the_same_bits_and_matches_the_oracle(dh, tokens, batches, masked):
    cfg = dict(n_blocks=1, d_model=2 * dh, n_heads=2, d_mlp=64, seq_len=tokens, batch=max(batches), mode="bf16")
    flat, blocks, x, dy1, dy2 = make_case(cfg, seed=3)
    x2 = x[:, ::-1].copy()
    lens = np.full(cfg["batch"], tokens, np.int32)
    if masked:
        lens = np.random.default_rng(5).integers(1, tokens + 1, cfg["batch"]).astype(np.int32)
        lens[:2] = (1, min(tokens, 33))
    dev = [to_dev(a) for a in (x, x2, dy1, dy2)]

    def run(b):
        print(f"[case] dh {dh} tokens {tokens} batch {b}", flush=True)
        c = gpu_cfg(dict(cfg, batch=b))
        params = to_dev(flat, B.param_dtype(c))
        X1, X2, dY1, dY2 = (a[:b].contiguous() for a in dev)
        kl = torch.from_numpy(lens[:b].copy()).cuda()
        if masked:
            Y1, Y2 = B.rev_stack_forward_masked(c, params, X1, X2, kl)
            res = B.rev_stack_backward_reprop_masked(c, params, Y1, Y2, kl, dY1, dY2, want_inputs=True)
        else:
            Y1, Y2 = B.rev_stack_forward(c, params, X1, X2)
            res = B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2, want_inputs=True)
        torch.cuda.synchronize()
        return Y1, Y2, res

    full = run(max(batches))
    for b in batches[:-1]:
        Y1, Y2, res = run(b)
        assert torch.equal(Y1, full[0][:b]) and torch.equal(Y2, full[1][:b]), b
        for k in ("dX1", "dX2", "X1", "X2"):
            assert torch.equal(res[k], full[2][k][:b]), (b, k)
    # the last, smallest run against the oracle
    b = batches[0]
    Y1, Y2, res = run(b)
    y1, y2 = Y1.cpu().numpy(), Y2.cpu().numpy()
    kl = lens[:b] if masked else None
    ref = O.stack_backward_reversible_chunked(y1, y2, blocks, 2, dy1[:b], dy2[:b], chunk=1, key_len=kl)
    compare_backward(dict(cfg, batch=b), res, ref, TOL["bf16"], what=f"dh {dh} tokens {tokens}")
    for i in range(b):
        oy = O.stack_forward(x[i:i + 1].astype(np.float64), x2[i:i + 1].astype(np.float64), blocks, 2, 1e-6,
                             key_len=None if kl is None else kl[i:i + 1])
        assert rel_err(y1[i:i + 1], oy[0]) <= TOL["bf16"] and rel_err(y2[i:i + 1], oy[1]) <= TOL["bf16"]
