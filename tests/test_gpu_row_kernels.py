"""GPU parity of the row kernels and of the decoding products where their layouts change: rows of less than a wavefront, of
one to four wavefronts and of more, fan-outs with and without a kernel of their own, sorted copies made from the sorted side
and from the source side, decoding tiles one, two and four wavefronts across with a ragged last tile."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return m


def _mlp_all(smoe, cfg, seed, backward=True):
    case = si.mlp_case(cfg, seed)
    ei, g, se, o, off = oracle_routing(case["logits"], cfg.k, cfg.E)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), cfg.k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, cfg.E)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    Y, buf = smoe.mlp_fwd(X, W1, W2, r, cfg.k, gg, cfg.act)
    g64 = oracle_gates_f32(g)
    args = [si.as_f64(case[n]) for n in ("X", "W1", "W2")]
    assert_close(Y, oracle.mlp_fwd(*args, ei, g64, cfg.act)["Y"], torch.bfloat16, "Y")
    if not backward:
        return
    grads = smoe.mlp_bwd(dY, X, W1, W2, r, cfg.k, gg, cfg.act, buf)
    ref = oracle.mlp_bwd(si.as_f64(case["dY"]), *args, ei, g64, cfg.act)
    for got, name in zip(grads, ("dX", "dW1", "dW2", "dgates")):
        assert_close(got, ref[name], torch.bfloat16, name)


# d_model / 8 chunks a row: 13 (16 lanes), 65 (two wavefronts), 129 (three), 193 (four), 257 (four, twice round)
@pytest.mark.parametrize("d_model", [104, 520, 1032, 1544, 2056])
@pytest.mark.parametrize("k,act", [(1, si.ACT_GELU), (2, si.ACT_SWIGLU), (3, si.ACT_GELU), (4, si.ACT_SWIGLU), (8, si.ACT_GELU)])
def test_row_kernels_in_the_mlp(smoe, d_model, k, act):
    print("rows", d_model, k, act, flush=True)
    _mlp_all(smoe, si.custom("rows", T=67, d_model=d_model, d_expert=136, E=9, k=k, act=act, dtype="bf16"), 71)


# numbers of slots with a kernel of their own (1 to 8), and above: batches of eight with and without rows left over
@pytest.mark.parametrize("k", [5, 6, 7, 9, 16, 19])
def test_row_kernels_for_every_number_of_slots(smoe, k):
    print("slots", k, flush=True)
    _mlp_all(smoe, si.custom("slots", T=37, d_model=104, d_expert=72, E=19, k=k, act=si.ACT_SWIGLU, dtype="bf16"), 79)


@pytest.mark.parametrize("k", [3, 4])
def test_sorted_copies_spread_from_the_source_rows(smoe, k):
    """The weight gradient of a product large enough for its operands to be spread, next to half of its rows (grouped)."""
    E, d = 5, 1024
    full = (24 << 20) // (2 * d) // k + 1
    for T in (full, full // 2):
        print("spread", T, k, flush=True)
        gen = torch.Generator(device="cuda").manual_seed(7)
        X, dY, W = (torch.randn(*s, generator=gen, device="cuda").bfloat16() for s in ((T, d), (T, d), (E, d, d)))
        ei, g = smoe.topk_gate(torch.randn(T, E, generator=gen, device="cuda"), k)
        r = smoe.route(ei, E)
        _, Yhat = smoe.plinear_fwd(X, W, r, k, g)
        _, dW, _ = smoe.plinear_bwd(dY, X, W, Yhat, r, k, g)
        for e in range(E):
            t, j = (ei == e).nonzero(as_tuple=True)
            ref = X[t].float().t() @ (dY[t].float() * g[t, j, None]).bfloat16().float()
            assert_close(dW[e], ref.cpu().numpy(), torch.bfloat16, f"dW[{e}]")


# wavefronts across a tile of the two products: 4 and 1, 2 and 2, 1 and 4 (64 experts, 256 compute units)
@pytest.mark.parametrize("d_model,d_expert", [(544, 1120), (1056, 544), (2080, 96)])
@pytest.mark.parametrize("act", [si.ACT_SWIGLU, si.ACT_GELU])
def test_decode_tiles_of_every_width(smoe, d_model, d_expert, act):
    print("decode", d_model, d_expert, act, flush=True)
    _mlp_all(smoe, si.custom("dec", T=40, d_model=d_model, d_expert=d_expert, E=64, k=8, act=act, dtype="bf16"), 73, backward=False)


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 7, 8, 9, 13])
@pytest.mark.parametrize("d_out", [264, 8200, 16392], ids=["four-shares", "two-shares", "one-share"])
def test_decode_contractions_of_every_remainder(smoe, steps, d_out):
    """Contractions of few 32-row steps, shared by four, two and one wavefronts: shares of no step, of fewer than are asked for
    ahead, and every remainder of the loop that keeps two in flight."""
    T, E, d_in = 70, 8, 32 * steps
    print("decode steps", steps, d_out, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(steps)
    X = torch.randn(T, d_in, generator=gen, device="cuda").bfloat16()
    W = (torch.randn(E, d_in, d_out, generator=gen, device="cuda") * 0.1).bfloat16()
    logits = torch.randn(T, E, generator=gen, device="cuda")
    logits[:40, 1] += 100.0                       # one expert with two row tiles
    ei, _ = smoe.topk_gate(logits, 1)
    r = smoe.route(ei, E)
    Y, _ = smoe.plinear_fwd(X, W, r, 1)
    for e in range(E):
        t = (ei[:, 0] == e).nonzero()[:, 0]
        if len(t):
            assert_close(Y[t], (X[t].float() @ W[e].float()).cpu().numpy(), torch.bfloat16, f"Y of expert {e}")
