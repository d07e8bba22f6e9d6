"""The attention layer's backward pass where the output projection's input-gradient product leaves dp, delta and the weighted rows
of Ohat in its epilogue and dQ is written in expert-sorted order (large layers take that route; the 256 x 256 tiles forced, all
do): segments and sequences that end inside a tile, several tile columns, an odd number of heads (the slabs of dp are even),
contractions that are and are not a multiple of 128, experts without tokens, k up to 8.  Every gradient against the oracle, and
against the route of the small layers, whose dp goes through bf16 rows of Yhat."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def smoe():
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    yield m
    m.set_kernel_mode(0)


@pytest.mark.parametrize("B,T,d_model,E,k,h,masked", [
    (1, 129, 264, 4, 2, 1, 0),       # one head: the second slab of a 256-column tile is empty
    (2, 111, 256, 3, 3, 3, 0),       # odd number of heads over two tile columns
    (1, 300, 136, 12, 8, 2, 3),      # k = 8, experts without tokens
    (3, 77, 648, 5, 4, 4, 0),        # contraction that ends inside a half-step, two tile columns
])
def test_every_gradient(smoe, B, T, d_model, E, k, h, masked):
    N, d_out = B * T, h * 128
    print("epilogue", B, T, d_model, E, k, h, masked, flush=True)
    gen = torch.Generator().manual_seed(91)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=gen) * std).bfloat16()
    X, dO = rnd(N, d_model), rnd(N, d_model)
    W_K, W_V = rnd(d_model, d_out, std=0.05), rnd(d_model, d_out, std=0.05)
    W_Q, W_O = rnd(E, d_model, d_out, std=0.05), rnd(E, d_out, d_model, std=0.05)
    logits = torch.randn(N, E, generator=gen)
    logits[:, E - masked:] = -1e30
    ei, g, _, _, _ = oracle_routing(logits, k, E)
    args = [t.cuda() for t in (X, W_K, W_V, W_Q, W_O)]

    def run(mode):
        smoe.set_kernel_mode(mode)
        gi, gg = smoe.topk_gate(logits.cuda(), k)
        r = smoe.route(gi, E)
        _, buf = smoe.momha_fwd(*args, r, k, gg, B, T, h, 128)
        return gi, smoe.momha_bwd(dO.cuda(), *args, r, k, gg, B, T, h, 128, buf)

    gi, got = run(4)
    assert np.array_equal(gi.cpu().numpy(), ei)
    small = run(0)[1]
    again = run(4)[1]
    ref = oracle.momha_bwd(si.as_f64(dO), *[si.as_f64(t) for t in (X, W_K, W_V, W_Q, W_O)], ei, oracle_gates_f32(g), B, T, h, 128)
    for i, name in enumerate(("dX", "dW_K", "dW_V", "dW_Q", "dW_O", "dgates")):
        assert_close(got[i].reshape(ref[name].shape), ref[name], BF, name)
        assert_close(small[i].reshape(ref[name].shape), ref[name], BF, name + " (small layers)")
        assert torch.equal(got[i], again[i]), name        # deterministic
