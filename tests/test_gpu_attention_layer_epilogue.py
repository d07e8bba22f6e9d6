"""The attention layer's backward pass where the output projection's input-gradient product leaves dp and the weighted rows of
Ohat in its epilogue and dQ is written in expert-sorted order (large layers take that route; the 256 x 256 tiles forced, all
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
        if mode == 4:
            buf.Yhat.fill_(float("nan"))         # only the other route reads it
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


@pytest.mark.parametrize("d_model", [256, 136])    # contractions that are and are not a multiple of 128
def test_several_tiles_per_block(smoe, d_model):
    """Every block of the output projection's product works through two tiles and more, with rows of dO everywhere: dX and dgates of
    tokens from every tile of every expert (sequences are independent, the oracle runs theirs), and every row of dW_O at sampled
    columns (column c depends on column c of dO only)."""
    B, T, E, k, h = 683, 3, 16, 8, 16
    N, d_out = B * T, h * 128
    print("epilogue, several tiles per block", d_model, flush=True)
    gen = torch.Generator().manual_seed(94)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=gen) * std).bfloat16()
    X, dO = rnd(N, d_model), rnd(N, d_model)
    W_K, W_V = rnd(d_model, d_out, std=0.06), rnd(d_model, d_out, std=0.06)
    W_Q, W_O = rnd(E, d_model, d_out, std=0.06), rnd(E, d_out, d_model, std=0.02)
    logits = torch.randn(N, E, generator=gen) + torch.linspace(1.0, -1.0, E)      # segments of different lengths
    ei, g, _, o, off = oracle_routing(logits, k, E)
    tiles = [(e, a) for e in range(E) for a in range(int(off[e]), int(off[e + 1]), 256)]
    assert len(tiles) * (d_out // 256) >= 2 * 256
    args = [t.cuda() for t in (X, W_K, W_V, W_Q, W_O)]
    smoe.set_kernel_mode(4)
    gi, gg = smoe.topk_gate(logits.cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    _, buf = smoe.momha_fwd(*args, r, k, gg, B, T, h, 128)
    buf.Yhat.fill_(float("nan"))                 # only the other route reads it
    got = smoe.momha_bwd(dO.cuda(), *args, r, k, gg, B, T, h, 128, buf)
    for t, name in zip(got, ("dX", "dW_K", "dW_V", "dW_Q", "dW_O", "dgates")):
        assert bool(torch.isfinite(t.float()).all()), f"{name} holds entries no kernel wrote"
    g64 = oracle_gates_f32(g)
    X64, dO64, K64, V64, Q64, O64 = (si.as_f64(t) for t in (X, dO, W_K, W_V, W_Q, W_O))
    rng = np.random.default_rng(7)
    rows = [int(rng.integers(a, min(a + 256, int(off[e + 1])))) for e, a in tiles]
    seqs = np.unique(o[rows] // k // T)
    S = (seqs[:, None] * T + np.arange(T)).ravel()
    ref = oracle.momha_bwd(dO64[S], X64[S], K64, V64, Q64, O64, ei[S], g64[S], len(seqs), T, h, 128)
    st = torch.from_numpy(S).cuda()
    assert_close(got[0][st], ref["dX"], BF, "dX (sequences from every tile)")
    assert_close(got[5].reshape(N, k)[st], ref["dgates"], BF, "dgates (sequences from every tile)")
    cols = np.sort(rng.choice(d_model, 6, replace=False))
    Ohat = oracle.momha_fwd(X64, K64, V64, Q64, O64[:, :, cols], ei, g64, B, T, h, 128)["Ohat"]
    upstream = (g64[:, :, None] * dO64[:, None, cols]).reshape(N * k, -1)
    dW_O = np.stack([Ohat[ei.ravel() == e].T @ upstream[ei.ravel() == e] for e in range(E)])
    got_cols = got[4][:, :, torch.from_numpy(cols).cuda()]
    assert_close(got_cols.transpose(1, 2), dW_O.transpose(0, 2, 1), BF, "dW_O (sampled columns, every row)")


@pytest.mark.parametrize("mode,in_epilogue", [(0, True), (4, True), (3, False)])
def test_which_layers_take_the_epilogue(smoe, mode, in_epilogue):
    """A layer large enough to take it by itself.  Only the route of the small layers reads the saved Yhat, so NaN there show in
    dgates, and in nothing else, exactly where that route is taken: with the 128 x 256 tiles forced, which the epilogue does not fit."""
    B, T, d_model, E, k, h = 8, 512, 512, 8, 8, 2
    N, d_out = B * T, h * 128
    assert N * k * d_model >= 16 << 20 and -(-N * k // 256) * -(-d_out // 256) * 2 >= 256
    print("route", mode, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(93)
    rnd = lambda *s, std=1.0: torch.empty(*s, dtype=BF, device="cuda").normal_(0.0, std, generator=gen)
    X, dO = rnd(N, d_model), rnd(N, d_model)
    args = [X, rnd(d_model, d_out, std=0.05), rnd(d_model, d_out, std=0.05), rnd(E, d_model, d_out, std=0.05), rnd(E, d_out, d_model, std=0.05)]
    smoe.set_kernel_mode(mode)
    gi, gg = smoe.topk_gate(torch.empty(N, E, device="cuda").normal_(0.0, 1.0, generator=gen), k)
    r = smoe.route(gi, E)
    _, buf = smoe.momha_fwd(*args, r, k, gg, B, T, h, 128)
    want = smoe.momha_bwd(dO, *args, r, k, gg, B, T, h, 128, buf)
    buf.Yhat.fill_(float("nan"))
    got = smoe.momha_bwd(dO, *args, r, k, gg, B, T, h, 128, buf)
    for a, b in zip(got[:5], want[:5]):
        assert torch.equal(a, b)
    assert torch.equal(got[5], want[5]) if in_epilogue else bool(got[5].isnan().all())


@pytest.mark.parametrize("B,k,h", [(37, 4, 3), (150, 2, 2)])
@pytest.mark.parametrize("mode", [4, 0])
def test_a_softmax_row_of_one_key_has_no_score_gradient(smoe, mode, B, k, h):
    """Sequences of one position: P = 1, Ohat = V, so dP - delta is the difference of two fp32 sums of the same 128 products of the
    stored dOhat and V, whatever rounding dOhat went through: at most 2 * (128 + 16) * 2^-23 of the sum of their magnitudes, and
    dW_Q and dW_K at most that times the sums of magnitudes behind them (1.02: the bf16 roundings of dS, dQ and dK).  delta from
    dOhat before its rounding is off by 2^-9 of every product instead."""
    d_model, E = 264, 64
    d_out = h * 128
    print("one key", mode, B, k, h, flush=True)
    gen = torch.Generator().manual_seed(92)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=gen) * std).bfloat16()
    X, dO = rnd(B, d_model), rnd(B, d_model)
    W_K, W_V = rnd(d_model, d_out, std=0.06), rnd(d_model, d_out, std=0.06)
    W_Q, W_O = rnd(E, d_model, d_out, std=0.06), rnd(E, d_out, d_model, std=0.06)
    args = [t.cuda() for t in (X, W_K, W_V, W_Q, W_O)]
    smoe.set_kernel_mode(mode)
    gi, gg = smoe.topk_gate(torch.randn(B, E, generator=gen).cuda(), k)
    r = smoe.route(gi, E)
    _, buf = smoe.momha_fwd(*args, r, k, gg, B, 1, h, 128)
    got = smoe.momha_bwd(dO.cuda(), *args, r, k, gg, B, 1, h, 128, buf)
    K, V, Q = (si.as_f64(t.cpu()).reshape(B, -1, h, 128) for t in (buf.K, buf.V, buf.Q))
    ei, g, X64, dO64, WO64 = gi.cpu().numpy(), gg.cpu().numpy().astype(np.float64), si.as_f64(X), si.as_f64(dO), si.as_f64(W_O)
    unit = 2 * (128 + 16) * 2.0 ** -23 * 1.02 / np.sqrt(128)
    dK_max, dW_Q_max = np.zeros((B, h, 128)), np.zeros((E, d_model, d_out))
    for t in range(B):
        for j in range(k):
            dOhat = np.abs(g[t, j] * (WO64[ei[t, j]] @ dO64[t])).reshape(h, 128) * 1.02
            dS = unit * (dOhat * np.abs(V[t, 0])).sum(axis=1, keepdims=True)
            dK_max[t] += dS * np.abs(Q[t, j])
            dW_Q_max[ei[t, j]] += np.outer(np.abs(X64[t]), dS * np.abs(K[t, 0]))
    for i, bound, name in ((1, np.abs(X64).T @ dK_max.reshape(B, d_out), "dW_K"), (3, dW_Q_max, "dW_Q")):
        over = np.abs(si.as_f64(got[i].cpu())) / np.maximum(bound, 1e-300)
        print(name, "largest share of its bound", over.max(), flush=True)
        assert over.max() <= 1, name
    assert_close(got[2], X64.T @ _dv(ei, g, dO64, WO64, B, d_out), BF, "dW_V")


def _dv(ei, g, dO64, WO64, B, d_out):
    return np.stack([sum(g[t, j] * (WO64[ei[t, j]] @ dO64[t]) for j in range(ei.shape[1])) for t in range(B)]).reshape(B, d_out)
