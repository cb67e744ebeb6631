"""The bits of a sample (outputs, reconstructed inputs, input gradients) are the same alone and in batches of every size: all
tiles of the bf16 GEMMs sum the products of an output element in one order."""
import pytest
import torch

from paper_2306_09342_amd import binding as B

from parity_util import gpu_cfg, make_case, to_dev

pytestmark = pytest.mark.gpu

# name -> (stack, batches): the row counts put every GEMM of the block into tiles of every kind (32x32, 64x64, 64x128 in
# the ring and in two stages, 128x128, 160x128)
STACKS = {
    "width384": (dict(n_blocks=2, d_model=384, n_heads=6, d_mlp=1536, seq_len=197), (1, 2, 6, 16, 40, 90)),
    "width768": (dict(n_blocks=1, d_model=768, n_heads=12, d_mlp=3072, seq_len=197), (1, 3, 11, 16, 64)),
    "width1280": (dict(n_blocks=1, d_model=1280, n_heads=16, d_mlp=3840, seq_len=257), (1, 3, 10)),
    "ragged_width200": (dict(n_blocks=2, d_model=200, n_heads=5, d_mlp=808, seq_len=61), (1, 9, 40, 150)),
}


@pytest.mark.parametrize("name", list(STACKS))
def test_a_sample_has_the_same_bits_in_every_batch(name):
    shape, batches = STACKS[name]
    cfg = dict(shape, batch=max(batches), mode="bf16")
    flat, _, x, dy1, dy2 = make_case(cfg, seed=11)
    args = [to_dev(a) for a in (x, x[:, ::-1].copy(), dy1, dy2)]

    def run(b):
        print(f"[case] {name} batch {b}", flush=True)
        c = gpu_cfg(dict(cfg, batch=b))
        params = to_dev(flat, B.param_dtype(c))
        X1, X2, dY1, dY2 = (a[:b].contiguous() for a in args)
        Y1, Y2 = B.rev_stack_forward(c, params, X1, X2)
        out = [Y1, Y2]
        for res in (B.rev_stack_backward_reprop(c, params, Y1, Y2, dY1, dY2, want_inputs=True),
                    B.rev_stack_backward_pareprop(c, params, Y1, Y2, dY1, dY2, torch.cuda.Stream(), want_inputs=True)):
            out += [res[k] for k in ("dX1", "dX2", "X1", "X2")]
        torch.cuda.synchronize()
        return out

    full = run(max(batches))
    for b in batches[:-1]:
        for i, (got, want) in enumerate(zip(run(b), full)):
            assert torch.equal(got, want[:b]), (b, i)
