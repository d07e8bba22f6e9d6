"""The output projection's input-gradient product with dp and the weighted rows of Ohat in its epilogue, on the 128 x 256 tiles: the same
dp, dW_O and (through dOhat) gradients of Q, K and V as on the 256 x 256 tiles, whose sums run in the same order, bit for bit."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
GRID = 256


def _estimate(rows, experts, K, N, tm, stage, rest):
    tiles = int((rows / tm + 0.5) * experts * math.ceil(N / 256) + 0.5)
    return math.ceil(tiles / GRID) * (stage * math.ceil(K / 64) + rest)


@pytest.mark.parametrize("T,d_model,heads,E,k", [
    (8066, 1064, 4, 4, 2),      # one round
    (4033, 2048, 4, 4, 4),
    (5400, 1560, 6, 2, 2),      # three tiles across
    (16200, 1032, 4, 4, 2),     # two rounds
])
def test_same_as_the_large_tiles(T, d_model, heads, E, k):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    Tk, width = T * k, heads * 128
    # in the epilogue, and on the small tiles
    assert Tk * d_model >= 16 << 20 and math.ceil(Tk / 256) * math.ceil(width / 256) * 2 >= GRID
    assert _estimate(Tk / E, E, d_model, width, 128, 0.9, 4) < 0.95 * _estimate(Tk / E, E, d_model, width, 256, 1.5, 6)
    print("attention layer, small tiles", T, d_model, heads, E, k, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, std=1.0: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=gen)
    logits = torch.empty(T, E, device="cuda").normal_(generator=gen)
    ei, g = smoe.topk_gate(logits, k)
    r = smoe.route(ei, E)
    a = (normal(T, d_model), normal(d_model, width, std=d_model ** -0.5), normal(d_model, width, std=d_model ** -0.5),
         normal(E, d_model, width, std=d_model ** -0.5), normal(E, width, d_model, std=width ** -0.5), r, k, g, 1, T, heads, 128)
    dO = normal(T, d_model)
    _, buf = smoe.momha_fwd(*a)
    got = {}
    for mode in (0, 4):
        smoe.set_kernel_mode(mode)
        try:
            got[mode] = [t.clone() for t in smoe.momha_bwd(dO, *a, buf)]
        finally:
            smoe.set_kernel_mode(0)
    names = ("dX", "dW_K", "dW_V", "dW_Q", "dW_O", "dgates")
    for n, x, y in zip(names, got[0], got[4]):
        assert bool(torch.isfinite(x.float()).all()), n
        if n != "dX":              # other products of dX may be cut differently by the shape of their tiles
            assert torch.equal(x, y), n
    # dp against the product it replaces, <dO, Yhat>: the weighted sum over a token's slots is <dO, O>
    O = smoe.plinear_fwd(buf.Ohat, a[4], r, 1, g, False, False)[0]
    want = (dO.double() * O.double()).sum(1)
    have = (got[0][5].double() * g.double()).sum(1)
    assert float((want - have).norm() / want.norm()) < 2e-2
