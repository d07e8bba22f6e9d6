"""GPU parity of the attention layer's key and value projections and their gradients where they run as one launch: sequence
lengths that end inside a tile, widths of less than and more than a tile, and every tile shape; plus the weights that are read
past the caches by launches with at most one tile row per expert."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, last_round_plan, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[0, 2, 3, 4], ids=["auto", "per-tile", "tiles128", "tiles256"])
def smoe(request):
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.set_kernel_mode(request.param)
    yield m
    m.set_kernel_mode(0)


@pytest.mark.parametrize("B,T,d_model,h", [(1, 129, 264, 1), (1, 257, 136, 3), (3, 111, 520, 2)])
def test_key_and_value_projections(smoe, B, T, d_model, h):
    E, k, N, d_out = 4, 2, B * T, h * 128
    print("pair", B, T, d_model, h, flush=True)
    gen = torch.Generator().manual_seed(5)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=gen) * std).bfloat16()
    X, dO = rnd(N, d_model), rnd(N, d_model)
    W_K, W_V = rnd(d_model, d_out, std=0.05), rnd(d_model, d_out, std=0.05)
    W_Q, W_O = rnd(E, d_model, d_out, std=0.05), rnd(E, d_out, d_model, std=0.05)
    logits = torch.randn(N, E, generator=gen)
    ei, g, _, _, _ = oracle_routing(logits, k, E)
    gi, gg = smoe.topk_gate(logits.cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    args = [t.cuda() for t in (X, W_K, W_V, W_Q, W_O)]
    O, buf = smoe.momha_fwd(*args, r, k, gg, B, T, h, 128)
    dX, dW_K, dW_V, _, _, _ = smoe.momha_bwd(dO.cuda(), *args, r, k, gg, B, T, h, 128, buf)
    ref_args = [si.as_f64(t) for t in (X, W_K, W_V, W_Q, W_O)]
    g64 = oracle_gates_f32(g)
    ref = oracle.momha_fwd(*ref_args, ei, g64, B, T, h, 128)
    gref = oracle.momha_bwd(si.as_f64(dO), *ref_args, ei, g64, B, T, h, 128)
    bf = torch.bfloat16
    for got, want, name in ((buf.K, ref["K"], "K"), (buf.V, ref["V"], "V"), (O, ref["O"], "O"), (dX, gref["dX"], "dX"),
                            (dW_K, gref["dW_K"], "dW_K"), (dW_V, gref["dW_V"], "dW_V")):
        assert_close(got.reshape(want.shape), want, bf, name)


@pytest.mark.parametrize("mode", [3, 4], ids=["tiles128", "tiles256"])
@pytest.mark.parametrize("d_model,h,product", [(2840, 1, "forward"), (2816, 1, "forward"), (264, 22, "dX")])
def test_key_and_value_products_with_a_split_contraction(mode, d_model, h, product):
    """Both projections (their input gradients) in one launch whose contraction is cut into chunks: partial tiles of two segments,
    added and stored by the second kernel to the right one's output."""
    import paper_2403_08245_amd as m
    B, T, E, k, N, d_out = 1, 200, 3, 2, 200, h * 128
    K, width = (d_model, d_out) if product == "forward" else (d_out, d_model)
    tile = 128 if mode == 3 else 256
    whole, rest, chunks = last_round_plan([N, N], tile, width, K, mode == 4 and K % 128 == 0)
    assert whole == 0 and chunks == 4, (whole, rest, chunks)
    print("pair split", d_model, h, mode, flush=True)
    gen = torch.Generator().manual_seed(6)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=gen) * std).bfloat16()
    X, dO = rnd(N, d_model), rnd(N, d_model)
    W_K, W_V = rnd(d_model, d_out, std=0.02), rnd(d_model, d_out, std=0.02)
    W_Q, W_O = rnd(E, d_model, d_out, std=0.02), rnd(E, d_out, d_model, std=0.02)
    logits = torch.randn(N, E, generator=gen)
    ei, g, _, _, _ = oracle_routing(logits, k, E)
    gi, gg = m.topk_gate(logits.cuda(), k)
    r = m.route(gi, E)
    args = [t.cuda() for t in (X, W_K, W_V, W_Q, W_O)]
    m.set_kernel_mode(mode)
    try:
        _, buf = m.momha_fwd(*args, r, k, gg, B, T, h, 128)
        dX = m.momha_bwd(dO.cuda(), *args, r, k, gg, B, T, h, 128, buf)[0]
        torch.cuda.synchronize()
    finally:
        m.set_kernel_mode(0)
    ref_args = [si.as_f64(t) for t in (X, W_K, W_V, W_Q, W_O)]
    bf = torch.bfloat16
    assert_close(buf.K, ref_args[0] @ ref_args[1], bf, "K")
    assert_close(buf.V, ref_args[0] @ ref_args[2], bf, "V")
    gref = oracle.momha_bwd(si.as_f64(dO), *ref_args, ei, oracle_gates_f32(g), B, T, h, 128)
    assert_close(dX, gref["dX"], bf, "dX")


def test_weights_read_past_the_caches(smoe):
    """More weights than the last-level cache holds and at most one tile of rows per expert, empty experts among them."""
    E, k, T, d_in, d_out = 24, 1, 1000, 1032, 5640
    gen = torch.Generator(device="cuda").manual_seed(9)
    X = torch.randn(T, d_in, generator=gen, device="cuda").bfloat16()
    W = (torch.randn(E, d_in, d_out, generator=gen, device="cuda") * 0.03).bfloat16()
    assert W.numel() * 2 > 256 << 20 and T * k <= 128 * E and T * k > 32 * E
    logits = torch.randn(T, E, generator=gen, device="cuda")
    logits[:, 5:8] = -100.0
    ei, _ = smoe.topk_gate(logits, k)
    r = smoe.route(ei, E)
    Y, _ = smoe.plinear_fwd(X, W, r, k)
    for e in range(E):
        t = (ei[:, 0] == e).nonzero()[:, 0]
        assert len(t) or 5 <= e < 8
        if len(t):
            assert_close(Y[t], (X[t].float() @ W[e].float()).cpu().numpy(), torch.bfloat16, f"Y of expert {e}")


@pytest.mark.parametrize("T,d_in", [(1000, 1032), (700, 1056)], ids=["tiles", "decode"])
def test_weights_of_a_popular_expert_among_those_read_past_the_caches(smoe, T, d_in):
    """As above with half of the rows on one expert: its several tiles read its weights through the caches, the others' one
    tile past them, in the same launch."""
    E, k, d_out = 24, 1, 5640
    print("popular", T, d_in, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    X = torch.randn(T, d_in, generator=gen, device="cuda").bfloat16()
    W = (torch.randn(E, d_in, d_out, generator=gen, device="cuda") * 0.03).bfloat16()
    assert W.numel() * 2 > 256 << 20 and (T > 32 * E or d_in % 32 == 0)
    logits = torch.randn(T, E, generator=gen, device="cuda")
    logits[:, 5:8] = -100.0
    logits[::2, 3] = 100.0
    ei, _ = smoe.topk_gate(logits, k)
    r = smoe.route(ei, E)
    Y, _ = smoe.plinear_fwd(X, W, r, k)
    for e in range(E):
        t = (ei[:, 0] == e).nonzero()[:, 0]
        assert len(t) >= T // 2 if e == 3 else len(t) <= 128
        if len(t):
            assert_close(Y[t], (X[t].float() @ W[e].float()).cpu().numpy(), torch.bfloat16, f"Y of expert {e}")
