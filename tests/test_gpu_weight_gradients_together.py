"""Both weight gradients of the MLP in one launch, taken where that saves a round of tiles: widths that end inside a tile on every
side, segments of different lengths and none, the routing-weighted copy of dY (SwiGLU) and the weighted hidden rows (GELU, narrower
than the model), one slot per token (sorted copies gathered) and two (spread).  Every entry of every gradient against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu
GRID, TB = 256, 256


@pytest.mark.parametrize("T,d_model,d_expert,E,k,act", [
    (140, 1032, 1416, 9, 1, si.ACT_SWIGLU),
    (70, 1288, 1032, 9, 2, si.ACT_GELU),
    (60, 1032, 1288, 9, 2, si.ACT_NONE),
])
def test_every_entry(T, d_model, d_expert, E, k, act):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    d_h = smoe.hidden_width(act, d_expert)
    tiles = lambda m, n: E * -(-m // TB) * -(-n // TB)
    rounds = lambda t: -(-t // GRID)
    first, further = tiles(d_expert, d_model), tiles(d_model, d_h)
    assert min(first, further) * 2 > GRID and rounds(first + further) < rounds(first) + rounds(further)   # the launch under test is taken
    cfg = si.custom("together", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=act, dtype="bf16", masked_experts=1)
    case = si.mlp_case(cfg, 97)
    ei, g, _, _, _ = oracle_routing(case["logits"], k, E)
    print("together", T, d_model, d_expert, E, k, act, np.bincount(ei.ravel(), minlength=E).tolist(), flush=True)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    _, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, act)
    assert buf.Yhat is None          # the persistent kernels take these widths
    got = smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf)
    ref = oracle.mlp_bwd(si.as_f64(case["dY"]), *[si.as_f64(case[n]) for n in ("X", "W1", "W2")], ei, oracle_gates_f32(g), act)
    for t, nm in zip(got, ("dX", "dW1", "dW2", "dgates")):
        assert_close(t, ref[nm], torch.bfloat16, nm)
