"""bf16 results that must not depend on which tile a GEMM launch takes.

* The bits of a sample (outputs, reconstructed inputs, input gradients) are the same alone and in batches of every size:
  all tiles sum the products of an output element in one order.
* Widths that are no multiple of 32 evaluate GELU and its derivative in the erf form, whose error is far below the bf16
  rounding of the stored value."""
import math

import numpy as np
import pytest
import torch

from paper_2306_09342_amd import binding as B

from parity_util import gpu_cfg, make_case, to_dev

pytestmark = pytest.mark.gpu

T_BFC1, T_WFC2 = 9, 10          # positions in the packed parameter vector

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


def _gelu(x):
    cdf = np.asarray([0.5 * math.erfc(-v / math.sqrt(2.0)) for v in x])
    return x * cdf, cdf + x * np.exp(-0.5 * x * x) / math.sqrt(2.0 * math.pi)


# (width, heads, tokens, batch): 32x32, 64x64 and 128x128 tiles
@pytest.mark.parametrize("width,heads,tokens,batch", [(40, 1, 3, 1), (72, 1, 100, 64), (72, 1, 100, 200)])
def test_gelu_of_widths_off_the_multiples_of_32_is_exact_to_bf16(width, heads, tokens, batch):
    """fc1's weight is zero and its bias h a ramp over [-6, 6], fc2 the identity: Y2 - X2 is the stored bf16 GELU of h, and
    with dY2 = 1 the gradient of h is the derivative, summed over the tokens."""
    c = B.make_cfg(n_blocks=1, d_model=width, n_heads=heads, d_mlp=width, seq_len=tokens, batch=batch, mode="bf16")
    h = torch.linspace(-6.0, 6.0, width).to(torch.bfloat16)
    params = torch.zeros(B.rev_stack_param_count(c), device="cuda", dtype=torch.bfloat16)

    def put(tensor, value):
        off, n = B.rev_stack_param_offset(c, 0, tensor)
        params[off:off + n] = value.reshape(-1).to(params)

    put(T_BFC1, h)
    put(T_WFC2, torch.eye(width))
    zero = torch.zeros(batch, tokens, width, device="cuda")
    Y1, Y2 = B.rev_stack_forward(c, params, zero, zero)
    res = B.rev_stack_backward_reprop(c, params, Y1, Y2, zero, torch.ones_like(zero))
    torch.cuda.synchronize()
    value, slope = _gelu(h.double().numpy())
    # half a bf16 step (at most 2^-8 of the value), and a few float32 steps of erff's 1 + erf(x), which cancels for negative x
    err = np.abs(Y2.double().cpu().numpy() - value)
    assert (err <= np.abs(value) / 256 * 1.01 + 1e-6).all(), err.max()
    off, n = B.rev_stack_param_offset(c, 0, T_BFC1)
    got = res["dparams"][off:off + n].double().cpu().numpy() / (tokens * batch)
    # float32 sums of equal terms: strips of up to 64 rows, then up to 313 strips one after the other, 2^-24 per addition
    assert np.abs(got - slope).max() <= (64 + 313) * 1.13 * 2.0 ** -24, np.abs(got - slope).max()
