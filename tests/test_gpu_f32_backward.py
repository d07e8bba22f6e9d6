"""The fp32 backward pass in one launch per ParallelLinear: every combination of its parts (input gradient, weight gradient,
routing-weight gradient), around the 64-row and 64-column tiles, with contractions of one and several 32-deep steps, empty and
long segments; and outputs that lie over an input which only an earlier part reads, where the parts must stay launches of
their own.  Against the fp64 oracle at 1e-5 of the largest entry: sums of up to a few hundred fp32 terms."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu
F = torch.float32


@pytest.fixture(scope="module")
def smoe():
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return m


@pytest.mark.parametrize("T,d_in,d_out,E,k,grouped_in,grouped_out,with_p", [
    (1, 4, 4, 3, 1, False, False, True),            # one row, two experts without any
    (65, 32, 68, 1, 1, True, False, False),         # one segment of a tile and one row, a single step
    (130, 68, 100, 4, 2, False, False, True),       # steps 2 and 3 deep, k-sum of dX
    (130, 100, 36, 4, 3, False, True, False),       # grouped upstream rows
    (193, 260, 132, 40, 2, True, False, True),      # many short segments, five steps
])
@pytest.mark.parametrize("need_dX,need_dW", [(True, True), (True, False), (False, True)])
def test_parts_in_one_launch(smoe, T, d_in, d_out, E, k, grouped_in, grouped_out, with_p, need_dX, need_dW):
    c = si.plinear_case(T, d_in, d_out, E, k, "f32", seed=81, x_rows=T * k if grouped_in else T)
    ei, g, se, o, off = oracle_routing(c["logits"], k, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    g64, gg = oracle_gates_f32(g), torch.from_numpy(g.astype(np.float32)).cuda()
    fan = 1 if grouped_in else k
    dY = c["dY_T"] if with_p else c["dY_Tk"]
    print("f32 backward", T, d_in, d_out, E, k, grouped_in, grouped_out, with_p, need_dX, need_dW, flush=True)
    X, W = c["X"].cuda(), c["W"].cuda()
    _, Yhat = smoe.plinear_fwd(X, W, r, fan, gg if with_p else None, grouped_in, grouped_out)
    dX, dW, dg = smoe.plinear_bwd(dY.cuda(), X, W, Yhat, r, fan, gg if with_p else None, grouped_in, grouped_out, need_dX, need_dW)
    ref = oracle.plinear_bwd(si.as_f64(dY), si.as_f64(c["X"]), si.as_f64(c["W"]), se, o, fan, g64 if with_p else None, grouped_in, grouped_out)
    for got, want, name in ((dX, ref[0], "dX"), (dW, ref[1], "dW"), (dg, ref[2], "dgates")):
        if got is not None:
            assert_close(got, want, F, name)
    assert (dX is not None) == need_dX and (dW is not None) == need_dW and (dg is not None) == with_p


@pytest.mark.parametrize("out,over", [("dX", "X"), ("dX", "Yhat"), ("dW", "Yhat")])
def test_outputs_over_inputs_of_earlier_parts(smoe, out, over):
    """dX over X (the weight gradient reads X first), dX or dW over Yhat (the row dots read it first)."""
    T, d, E = 192, 96, 2
    c = si.plinear_case(T, d, d, E, 1, "f32", seed=82)
    ei, g, _, _, _ = oracle_routing(c["logits"], 1, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    gates = torch.from_numpy(g.astype(np.float32)).cuda() * 0.5
    X, W, dY = c["X"].cuda(), c["W"].cuda(), c["dY_T"].cuda()
    _, Yhat = smoe.plinear_fwd(X, W, r, 1, gates)
    want = smoe.plinear_bwd(dY, X, W, Yhat, r, 1, gates)
    inputs = {"X": X.clone(), "Yhat": Yhat.clone()}
    dX, dW, dg = torch.empty_like(X), torch.empty_like(W), torch.empty_like(gates)
    if out == "dX":
        dX = inputs[over]
    else:
        dW = inputs[over].view_as(W)
    nb = smoe.lib.smoe_plinear_bwd_workspace_bytes(smoe.F32, T, d, d, T, 1, 1, 0, 0)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    rc = r.c()
    p = lambda t: t.data_ptr()
    assert smoe.lib.smoe_plinear_bwd(smoe.ctx(), smoe._stream(), smoe.F32, p(dY), p(inputs["X"]), T, d, p(W), d, p(inputs["Yhat"]), ctypes.byref(rc), 1,
                                     p(gates), 1, 0, 0, p(dX), p(dW), p(dg), p(ws), nb) == 0
    for got, ref, name in zip((dX, dW, dg), want, ("dX", "dW", "dgates")):
        assert torch.equal(got, ref), name


@pytest.mark.parametrize("out", ["dX over X", "dW2 over Yhat"])
def test_mlp_outputs_over_inputs_of_earlier_parts(smoe, out):
    """The whole MLP with k = 1: dX over X (dW1 reads X first), dW2 over the saved Yhat (the row dots read it first)."""
    E, d_model, d_expert = 2, 64, 96
    T = E * d_expert                     # dW2 is as large as Yhat
    cfg = si.custom("over", T=T, d_model=d_model, d_expert=d_expert, E=E, k=1, act=si.ACT_GELU, dtype="f32")
    case = si.mlp_case(cfg, 84)
    ei, g, _, _, _ = oracle_routing(case["logits"], 1, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    gates = torch.from_numpy(g.astype(np.float32)).cuda() * 0.5
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    _, buf = smoe.mlp_fwd(X, W1, W2, r, 1, gates, cfg.act)
    want = [t.clone() for t in smoe.mlp_bwd(dY, X, W1, W2, r, 1, gates, cfg.act, buf)]
    if out == "dX over X":
        buf.dX = X
    else:
        buf.dW2 = buf.Yhat.view(E, d_expert, d_model)
    got = smoe.mlp_bwd(dY, X, W1, W2, r, 1, gates, cfg.act, buf)
    for a, b, name in zip(got, want, ("dX", "dW1", "dW2", "dgates")):
        assert torch.equal(a, b), name


def test_more_blocks_than_one_launch_takes(smoe):
    """66 million rows of four: the input gradient and the row dots are each a launch the runtime accepts (under 2^32 threads), together
    they are not.  Four fp32 terms a sum."""
    Tk, d = 66_000_000, 4
    assert -(-Tk // 4) * 256 < 2 ** 32 < (-(-Tk // 4) + -(-Tk // 64) + 1) * 256
    print("f32 backward", Tk, "rows", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(83)
    rnd = lambda *s: torch.empty(*s, device="cuda").normal_(0.0, 1.0, generator=gen)
    X, Yhat, dY, W, gates = rnd(Tk, d), rnd(Tk, d), rnd(Tk, d), rnd(1, d, d), rnd(Tk, 1)
    o = torch.arange(Tk, dtype=torch.int32, device="cuda")
    r = smoe.Routing(torch.zeros_like(o), o, torch.tensor([0, Tk], dtype=torch.int32, device="cuda"), Tk, 1)
    dX, dW, dg = smoe.plinear_bwd(dY, X, W, Yhat, r, 1, gates, need_dW=False)
    assert dW is None
    assert torch.allclose(dg, (dY * Yhat).sum(1, keepdim=True), rtol=1e-5, atol=1e-5)
    assert torch.allclose(dX, gates * (dY @ W[0].t()), rtol=1e-5, atol=2e-5)
