"""Both weight gradients of the MLP in one launch, taken where that saves a round of tiles: widths that end inside a tile on every
side, segments of different lengths and none, the routing-weighted copy of dY (SwiGLU) and the weighted hidden rows (GELU, narrower
than the model), one slot per token (sorted copies gathered) and two (spread).  Segments of a few dozen rows: every entry of every
gradient against the oracle.  Segments of several groups of 128 rows: the oracle at hidden units of every tile, for every expert.  And
dW1 over the saved H, which the other launch order reads first."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu
GRID, TB = 256, 256


def _taken(smoe, d_model, d_expert, E, act):
    """Is the launch under test taken?"""
    tiles = lambda m, n: E * -(-m // TB) * -(-n // TB)
    rounds = lambda t: -(-t // GRID)
    first, further = tiles(d_expert, d_model), tiles(d_model, smoe.hidden_width(act, d_expert))
    return min(first, further) * 2 > GRID and rounds(first + further) < rounds(first) + rounds(further)


@pytest.mark.parametrize("T,d_model,d_expert,E,k,act", [
    (140, 1032, 1416, 9, 1, si.ACT_SWIGLU),
    (70, 1288, 1032, 9, 2, si.ACT_GELU),
    (60, 1032, 1288, 9, 2, si.ACT_NONE),
])
def test_every_entry(T, d_model, d_expert, E, k, act):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    assert _taken(smoe, d_model, d_expert, E, act)
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


# tokens per set of experts (one expert each for k = 1): segments of one to five groups of 128 rows, a few rows past a multiple of 128, whole
# multiples, a handful, none
ONE = {(0,): 517, (1,): 261, (2,): 130, (3,): 128, (4,): 256, (5,): 33, (7,): 3, (8,): 97}
TWO = {(0, 1): 261, (0, 2): 130, (0, 3): 129, (4, 8): 223, (4, 5): 33, (3, 7): 3}


@pytest.mark.parametrize("tokens,d_model,d_expert,act", [(ONE, 1032, 1416, si.ACT_SWIGLU), (TWO, 1288, 1032, si.ACT_GELU), (TWO, 1032, 1416, si.ACT_SWIGLU)])
def test_long_segments(tokens, d_model, d_expert, act):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    E, k, T = 9, len(next(iter(tokens))), sum(tokens.values())
    assert _taken(smoe, d_model, d_expert, E, act) and T * k * d_model * 2 <= 64 << 20
    cfg = si.custom("together-long", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=act, dtype="bf16")
    case = si.mlp_case(cfg, 98)
    logits = case["logits"] * 0.1
    where = np.random.default_rng(98).permutation(T)
    for experts, lo in zip(tokens, np.cumsum([0] + list(tokens.values()))):
        for e in experts:
            logits[where[lo:lo + tokens[experts]], e] += 8.0
    ei, g, _, o, off = oracle_routing(logits, k, E)
    loads = np.diff(off)
    print("together, long segments", T, d_model, d_expert, k, act, loads.tolist(), flush=True)
    assert loads.max() > 512 and loads.min() == 0 and any(128 < n and 0 < n % 128 <= 8 for n in loads) and any(n and n % 128 == 0 for n in loads)
    gi, gg = smoe.topk_gate(logits.cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    _, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, act)
    dX, dW1, dW2, dg = smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf)
    g64 = oracle_gates_f32(g)
    args = [si.as_f64(case[n]) for n in ("dY", "X", "W1", "W2")]
    rng = np.random.default_rng(4)
    units = np.concatenate([np.sort(rng.choice(np.arange(c, min(c + TB, d_expert)), 3, replace=False)) for c in range(0, d_expert, TB)])
    ut = torch.from_numpy(units).cuda()
    cols = [ut] + ([ut + d_expert] if act == si.ACT_SWIGLU else [])
    for e in range(E):
        assert_close(torch.stack([dW1[e][:, c].T for c in cols], 1), oracle.mlp_dW1_cols(*args, ei, g64, act, e, units), torch.bfloat16, f"dW1[{e}]")
        assert_close(dW2[e][ut], oracle.mlp_dW2_rows(*args, ei, g64, act, e, units), torch.bfloat16, f"dW2[{e}]")
    for n, t in (("dX", dX), ("dW1", dW1), ("dW2", dW2), ("dgates", dg)):
        assert bool(torch.isfinite(t.float()).all()), f"{n} holds entries no kernel wrote"
    if act == si.ACT_SWIGLU:             # the route that reads the saved H for dW2
        want = [t.clone() for t in (dX, dW1, dW2, dg)]
        over = torch.empty_like(buf.dW1)
        saved = over.view(-1)[:buf.H.numel()].view_as(buf.H)
        saved.copy_(buf.H)
        buf.dW1, buf.H = over, saved
        for a, b, n in zip(smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf), want, ("dX", "dW1", "dW2", "dgates")):
            assert torch.equal(a, b), n + " (dW1 over the saved H)"
