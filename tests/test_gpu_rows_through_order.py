"""groupXTY with rows of X, of dY or of both read through the order indices, against the same product of sorted copies, bit for bit (the
sums run in the same order): segments of one row up to several stages of 64 with a remainder, whole stages, none, several rounds of
tiles, and segments cut along their rows; fan-outs with and without an exact reciprocal; widths that end inside a tile.  Token 0
holds infinities: only its experts may see them, although lanes past a segment's end have index 0 at hand.  And outputs that lie over
the rows, for which sorted copies stand in."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _problem(loads, k, d_in, d_out, seed):
    """Tokens whose k slots fall on experts so that expert e gets loads[e] rows."""
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    rng = np.random.default_rng(seed)
    slots = rng.permutation(np.repeat(np.arange(len(loads), dtype=np.int32), loads))
    T, E = len(slots) // k, len(loads)
    r = smoe.route(torch.from_numpy(slots.reshape(T, k)).cuda(), E)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    print("rows through order", loads, k, d_in, d_out, flush=True)
    return smoe, r, slots, normal(T, d_in), normal(E, d_in, d_out), normal(T * k, d_out)


def _same(a, b, what):
    assert torch.equal(a.view(torch.int16), b.view(torch.int16)), what


@pytest.mark.parametrize("loads,k,d_in,d_out", [
    ([1, 63, 64, 65, 0, 127, 128, 129, 191, 193, 3], 1, 264, 520),
    ([1, 63, 64, 65, 0, 127, 128, 129, 191, 193, 3], 2, 1032, 248),
    ([5, 0, 255, 257, 640, 1, 4], 7, 256, 776),
    ([33, 95, 160, 224, 0, 64], 8, 2048, 2568),          # 6 x 88 tiles: more than two a block
    ([3100, 3083], 3, 264, 264),                         # eight tiles: cut along the rows
])
def test_same_as_sorted_copies(loads, k, d_in, d_out):
    smoe, r, slots, X, W, dY = _problem(loads, k, d_in, d_out, 5)
    X[0], dY[0] = float("inf"), float("inf")
    Xg, dYg = smoe.group(X, r, k), smoe.group(dY, r, 1)
    dXg, want, _ = smoe.plinear_bwd(dYg, Xg, W, None, r, 1, None, True, True)
    dX_want, _, _ = smoe.plinear_bwd(dYg, X, W, None, r, k, None, False, True, need_dW=False)
    others = torch.from_numpy(np.setdiff1d(np.arange(len(loads)), slots[:k])).cuda().long()
    assert bool(torch.isfinite(want[others].float()).all())
    dX, dW, _ = smoe.plinear_bwd(dYg, X, W, None, r, k, None, False, True)
    _same(dW, want, "dW, X through the order indices")
    _same(dX, dX_want, "dX, X through the order indices")
    dX, dW, _ = smoe.plinear_bwd(dY, Xg, W, None, r, 1, None, True, False)
    _same(dW, want, "dW, dY through the order indices")
    _same(dX, dXg, "dX, dY through the order indices")
    dX, dW, _ = smoe.plinear_bwd(dY, X, W, None, r, k, None, False, False)
    _same(dW, want, "dW, both through the order indices")
    _same(dX, dX_want, "dX, both through the order indices")


@pytest.mark.parametrize("over", ["dW over X", "dW over dY", "dX over dY"])
def test_outputs_over_the_rows(over, monkeypatch):
    loads, d = [70, 0, 131, 64, 1], 264
    smoe, r, _, X, W, dY = _problem(loads, 1, d, d, 6)
    dX_want, dW_want, _ = smoe.plinear_bwd(dY, X, W, None, r, 1)
    place = W if over.startswith("dW") else X
    mem = torch.empty_like(place)
    rows = mem.view(-1)[:X.numel()].view_as(X)
    src = X if over.endswith("X") else dY
    rows.copy_(src)
    monkeypatch.setattr(smoe, "_like", lambda t: mem if t is place else torch.empty_like(t))
    args = (dY, rows) if src is X else (rows, X)
    dX, dW, _ = smoe.plinear_bwd(args[0], args[1], W, None, r, 1)
    _same(dX, dX_want, "dX, " + over)
    _same(dW, dW_want, "dW, " + over)


def _mlp(T, d_model, d_expert, E, k, seed):
    import oracle
    import paper_2403_08245_amd as smoe
    import smoe_inputs as si
    from helpers import oracle_gates_f32, oracle_routing
    cfg = si.custom("weighted-hidden", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=si.ACT_SWIGLU, dtype="bf16", masked_experts=1)
    case = si.mlp_case(cfg, seed)
    ei, g, _, _, _ = oracle_routing(case["logits"], k, E)
    print("weighted hidden rows", T, d_model, d_expert, E, k, np.bincount(ei.ravel(), minlength=E).tolist(), flush=True)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    r = smoe.route(gi, E)
    _, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, si.ACT_SWIGLU)
    assert buf.Yhat is None          # the persistent kernels take these widths
    ref = oracle.mlp_bwd(si.as_f64(case["dY"]), *[si.as_f64(case[n]) for n in ("X", "W1", "W2")], ei, oracle_gates_f32(g), si.ACT_SWIGLU)
    return smoe, si, r, gg, X, W1, W2, dY, buf, ref


def _check(smoe, si, got, ref):
    from helpers import assert_close
    for t, nm in zip(got, ("dX", "dW1", "dW2", "dgates")):
        assert_close(t, ref[nm], torch.bfloat16, nm)


@pytest.mark.parametrize("mode", [3, 4], ids=["tiles128", "tiles256"])
@pytest.mark.parametrize("T,d_model,d_expert,E,k", [(300, 264, 264, 5, 1), (131, 520, 136, 4, 2), (90, 1032, 776, 3, 3)])
def test_swiglu_weighted_hidden_rows(mode, T, d_model, d_expert, E, k):
    """dW2 from routing-weighted hidden rows that the fused SwiGLU derivative leaves, where they are no wider than the model."""
    smoe, si, r, gg, X, W1, W2, dY, buf, ref = _mlp(T, d_model, d_expert, E, k, 61)
    smoe.set_kernel_mode(mode)
    try:
        got = smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, si.ACT_SWIGLU, buf)
    finally:
        smoe.set_kernel_mode(0)
    _check(smoe, si, got, ref)


@pytest.mark.parametrize("over,rows", [("dW1", "X"), ("dW1", "dY"), ("dW2", "dY")])   # X is read for dW1 after dW2 is written
def test_weight_gradient_over_the_rows(over, rows):
    smoe, si, r, gg, X, W1, W2, dY, buf, ref = _mlp(131, 264, 136, 4, 2, 62)
    mem = torch.empty_like(getattr(buf, over))
    src = X if rows == "X" else dY
    place = mem.view(-1)[:src.numel()].view_as(src)
    place.copy_(src)
    setattr(buf, over, mem)
    got = smoe.mlp_bwd(dY if rows == "X" else place, place if rows == "X" else X, W1, W2, r, 2, gg, si.ACT_SWIGLU, buf)
    _check(smoe, si, got, ref)
