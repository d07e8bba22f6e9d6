"""GPU parity of the two tile shapes of the persistent scatter2scatter kernels (256 x 256 tiles with one block per compute
unit, 128 x 256 with two) where they can go wrong: contractions that end inside a half-step of 32, the shortest ones they
take, segments at and around the tile heights, outputs narrower than a tile, and launches whose last round is one tile per
compute unit, cuts its contraction into chunks (with an end inside a half-step and without), or both.  Every row is compared with the oracle; outputs and workspaces are poisoned
and guard-banded (conftest.py)."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, last_round_plan, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[3, 4], ids=["tiles128", "tiles256"])
def smoe(request):
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.set_kernel_mode(request.param)
    yield m
    m.set_kernel_mode(0)


def _rows_at_tile_edges(T, E, k):
    """Expert choices (k = 1) whose segments have 1, 127, 128, 129, 255, 256, 257 rows, none, and the rest."""
    assert k == 1
    sizes = [1, 127, 128, 129, 255, 256, 257, 0]
    ids = np.concatenate([np.full(n, e) for e, n in enumerate(sizes[:E - 1])] + [np.full(T - sum(sizes[:E - 1]), E - 1)])
    return np.random.default_rng(3).permutation(ids).astype(np.int32).reshape(T, 1)


# T, d_in, d_out, E, k
CASES = [
    pytest.param(1500, 72, 264, 9, 1, id="K72-edges"),               # three half-steps, the last with 8 elements
    pytest.param(1500, 200, 96, 9, 1, id="K200-N96-edges"),
    pytest.param(1500, 2056, 1032, 9, 1, id="K2056-edges"),          # last round of few tiles, contraction with a tail of 8
    pytest.param(700, 96, 72, 3, 2, id="K96-N72"),
    pytest.param(9000, 136, 1304, 5, 2, id="K136-N1304-rounds"),     # several tiles per block, 128-row and 256-row last rounds ragged
    pytest.param(8500, 2832, 520, 8, 2, id="K2832-N520"),
]


@pytest.mark.parametrize("T,d_in,d_out,E,k", CASES)
def test_plinear_every_row(smoe, T, d_in, d_out, E, k):
    c = si.plinear_case(T, d_in, d_out, E, k, "bf16", seed=51)
    ei, g, se, o, off = oracle_routing(c["logits"], k, E)
    if k == 1:
        ei = _rows_at_tile_edges(T, E, k)
        se, o, off = oracle.route(ei, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    assert np.array_equal(r.sorted_scattered_idxs.cpu().numpy(), o)
    td = torch.bfloat16
    X, W, dY = c["X"].cuda(), c["W"].cuda(), c["dY_Tk"].cuda()
    print("plinear", T, d_in, d_out, E, k, np.diff(off).tolist(), flush=True)
    cols = np.unique(np.concatenate([np.arange(0, d_out, 37), np.arange(max(0, d_out - 9), d_out)]))
    rows = np.unique(np.concatenate([np.arange(0, d_in, 41), np.arange(max(0, d_in - 9), d_in)]))
    X64, W64, dY64 = si.as_f64(c["X"]), si.as_f64(c["W"]), si.as_f64(c["dY_Tk"])
    for gout in (False, True):
        Y, _ = smoe.plinear_fwd(X, W, r, k, None, False, gout)
        Y_ref, _ = oracle.plinear_fwd(X64, W64[:, :, cols], se, o, k, None, False, gout)
        assert_close(Y[:, torch.from_numpy(cols).cuda()], Y_ref, td, f"Y grouped_out={gout}")
        dX, dW, _ = smoe.plinear_bwd(dY, X, W, None, r, k, None, False, gout)
        dX_ref, dW_ref, _ = oracle.plinear_bwd(dY64, X64[:, rows], W64[:, rows, :], se, o, k, None, False, gout)
        rt = torch.from_numpy(rows).cuda()
        assert_close(dX[:, rt], dX_ref, td, f"dX grouped_out={gout}")
        assert_close(dW[:, rt, :], dW_ref, td, f"dW grouped_out={gout}")
        for name, t in (("Y", Y), ("dX", dX), ("dW", dW)):
            assert bool(torch.isfinite(t.float()).all()), f"{name} holds entries no kernel wrote"


# Input gradients with partial-tile scratch (plinear_bwd): contraction d_out, output width d_in; tile rows, and what the last round
# must plan (whole tiles, leftover tiles, chunks), so that a case cannot silently stop splitting.
SPLIT_CASES = [
    # 89 half-steps, the last with 24 elements; all tiles are leftovers
    pytest.param(1500, 1032, 2840, 9, 128, (0, 75, 4), id="tiles128-K2840-edges"),
    pytest.param(1500, 1032, 2840, 9, 256, (0, 50, 4), id="tiles256-K2840-edges"),
    # a multiple of 128: chunks of the 256-row tiles are whole groups of four half-steps
    pytest.param(1500, 1032, 2816, 9, 128, (0, 75, 4), id="tiles128-K2816-edges"),
    pytest.param(1500, 1032, 2816, 9, 256, (0, 50, 4), id="tiles256-K2816-edges"),
    # one 128-row tile on every compute unit and a few left over for the free halves of the grid
    pytest.param(6700, 1032, 2840, 3, 128, (256, 14, 4), id="tiles128-K2840-whole-and-split"),
    # a full round of 256-row tiles before the split one
    pytest.param(8000, 2056, 2840, 3, 256, (0, 41, 4), id="tiles256-K2840-round-and-split"),
]


@pytest.mark.parametrize("T,d_in,d_out,E,tile,planned", SPLIT_CASES)
@pytest.mark.parametrize("grouped_in", [False, True])
def test_split_last_round_every_row(T, d_in, d_out, E, tile, planned, grouped_in):
    import paper_2403_08245_amd as smoe
    c = si.plinear_case(T, d_in, d_out, E, 1, "bf16", seed=53)
    ei = _rows_at_tile_edges(T, E, 1) if E == 9 else oracle_routing(c["logits"], 1, E)[0]
    se, o, off = oracle.route(ei, E)
    assert last_round_plan(np.diff(off), tile, d_in, d_out, tile == 256 and d_out % 128 == 0) == planned
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    X, W, dY = c["X"].cuda(), c["W"].cuda(), c["dY_Tk"].cuda()
    print("split", T, d_in, d_out, E, tile, grouped_in, np.diff(off).tolist(), flush=True)
    rows = np.unique(np.concatenate([np.arange(0, d_in, 101), np.arange(max(0, d_in - 9), d_in)]))
    smoe.set_kernel_mode(3 if tile == 128 else 4)
    try:
        dX, again = (smoe.plinear_bwd(dY, X, W, None, r, 1, None, grouped_in, False)[0] for _ in range(2))
    finally:
        smoe.set_kernel_mode(0)
    dX_ref, _, _ = oracle.plinear_bwd(si.as_f64(c["dY_Tk"]), si.as_f64(c["X"])[:, rows], si.as_f64(c["W"])[:, rows, :], se, o, 1, None, grouped_in, False)
    assert_close(dX[:, torch.from_numpy(rows).cuda()], dX_ref, torch.bfloat16, "dX")
    assert bool(torch.isfinite(dX.float()).all()), "dX holds entries no kernel wrote"
    assert torch.equal(dX, again)          # the chunks are added in a fixed order


@pytest.mark.parametrize("act", [si.ACT_GELU, si.ACT_SWIGLU])
@pytest.mark.parametrize("T,d_model,d_expert,E,k", [(400, 104, 136, 4, 2), (400, 200, 88, 3, 3), (900, 80, 528, 5, 1)])
def test_mlp_every_row_with_contractions_inside_a_half_step(smoe, T, d_model, d_expert, E, k, act):
    """Both products and all gradients with neither width a multiple of 32: activation and derivative epilogues, the
    routing-weight gradient, and both ways of forming dW2 (d_expert on either side of d_model)."""
    cfg = si.custom("tails", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=act, dtype="bf16")
    case = si.mlp_case(cfg, 61)
    ei, g, se, o, off = oracle_routing(case["logits"], k, E)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    print("mlp", T, d_model, d_expert, E, k, act, flush=True)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    Y, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, act)
    assert buf.Yhat is None          # the persistent kernels take these widths
    dX, dW1, dW2, dg = smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf)
    g64 = oracle_gates_f32(g)
    args = [si.as_f64(case[n]) for n in ("X", "W1", "W2")]
    ref = oracle.mlp_fwd(*args, ei, g64, act)
    gref = oracle.mlp_bwd(si.as_f64(case["dY"]), *args, ei, g64, act)
    for got, want, nm in ((Y, ref["Y"], "Y"), (dX, gref["dX"], "dX"), (dW1, gref["dW1"], "dW1"), (dW2, gref["dW2"], "dW2"),
                          (dg, gref["dgates"], "dgates")):
        assert_close(got, want, torch.bfloat16, nm)
