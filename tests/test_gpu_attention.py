"""GPU parity of the attention kernels and of the SMoE attention layer (Alg. 4) against the fp64 oracle."""
import ctypes
import sys

import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import TOL, oracle_gates_f32

pytestmark = pytest.mark.gpu


def _log(*a):
    print(*a, flush=True, file=sys.stderr)


@pytest.fixture(scope="module")
def smoe():
    import paper_2403_08245_amd as m
    return m


def _bf16(shape, seed, std=1.0):
    x = torch.randn(*shape, generator=torch.Generator().manual_seed(seed), dtype=torch.float32) * std
    return x.to(torch.bfloat16)


def _rel(got, ref):
    return np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-3)   # a lone position has an exactly zero dQ and dK


ATTN_SHAPES = [(1, 1, 1, 1), (2, 77, 3, 2), (1, 300, 4, 1), (3, 33, 1, 2), (1, 130, 5, 1), (1, 64, 16, 1)]


@pytest.mark.parametrize("B,T,G,h", ATTN_SHAPES)
def test_attention_forward(smoe, B, T, G, h):
    _log(f"attention fwd B={B} T={T} G={G} h={h}")
    Q, K, V = _bf16((B, T, G, h, 128), 1), _bf16((B, T, h, 128), 2), _bf16((B, T, h, 128), 3)
    O, L = smoe.attention_fwd(Q.cuda(), K.cuda(), V.cuda())
    Oref, Lref = oracle.attention_fwd(si.as_f64(Q), si.as_f64(K), si.as_f64(V))
    assert _rel(O.float().cpu().numpy().astype(np.float64), Oref) <= TOL[torch.bfloat16]
    assert np.abs(L.cpu().numpy() - Lref).max() <= 2e-2        # log-sum-exp of O(10) scores from bf16 products


@pytest.mark.parametrize("peak", [0, 1, 2, 3, 4, 5, 6, 7, 13, 30, 36])
def test_attention_peaked_scores(smoe, peak):
    """One key whose score exceeds all others by 113 (in units of the exponent, more than fp32's range holds), at every
    position modulo 8 and in either tile of 32 keys: from that key's token on, O is its value row and the log-sum-exp its
    score.  Scores are exact in fp32 (1280 / sqrt(128)); the log-sum-exp is then good to a few fp32 roundings of 163 (its
    value in exp2 units), 4e-5, and is compared at 1e-3."""
    _log(f"attention peaked key={peak}")
    B, T, G, h = 1, 40, 2, 1
    Q, K, V = torch.full((B, T, G, h, 128), 10.0).bfloat16(), torch.zeros(B, T, h, 128).bfloat16(), _bf16((B, T, h, 128), 3)
    K[:, peak] = 1.0
    dO = _bf16((B, T, G, h, 128), 4)
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    O, L = smoe.attention_fwd(Qd, Kd, Vd)
    f64 = lambda t: t.float().cpu().numpy().astype(np.float64)
    Oref, Lref = oracle.attention_fwd(si.as_f64(Q), si.as_f64(K), si.as_f64(V))
    assert np.isfinite(f64(O)).all() and np.isfinite(f64(L)).all()
    assert _rel(f64(O), Oref) <= TOL[torch.bfloat16]
    assert torch.equal(O.cpu()[:, peak:], V[:, peak].reshape(B, 1, 1, h, 128).expand(B, T - peak, G, h, 128))
    assert np.abs(f64(L) - Lref).max() <= 1e-3
    dQ, dK, dV = smoe.attention_bwd(dO.cuda(), Qd, Kd, Vd, O, L)
    rv = oracle.attention_bwd(si.as_f64(dO), si.as_f64(Q), si.as_f64(K), si.as_f64(V))[2]
    assert np.isfinite(f64(dQ)).all() and np.isfinite(f64(dK)).all()
    assert _rel(f64(dV), rv) <= TOL[torch.bfloat16]


@pytest.mark.parametrize("B,T,G,h", ATTN_SHAPES)
def test_attention_backward(smoe, B, T, G, h):
    _log(f"attention bwd B={B} T={T} G={G} h={h}")
    Q, K, V = _bf16((B, T, G, h, 128), 1), _bf16((B, T, h, 128), 2), _bf16((B, T, h, 128), 3)
    dO = _bf16((B, T, G, h, 128), 4)
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    O, L = smoe.attention_fwd(Qd, Kd, Vd)
    dQ, dK, dV = smoe.attention_bwd(dO.cuda(), Qd, Kd, Vd, O, L)
    rq, rk, rv = oracle.attention_bwd(si.as_f64(dO), si.as_f64(Q), si.as_f64(K), si.as_f64(V))
    for name, got, ref in (("dQ", dQ, rq), ("dK", dK, rk), ("dV", dV, rv)):
        err = _rel(got.float().cpu().numpy().astype(np.float64), ref)
        _log(f"  {name} rel err {err:.2e}")
        assert err <= TOL[torch.bfloat16], name


def _layer_case(seed, B, T, d_model, E, k, h):
    d_out = h * 128
    N = B * T
    X = _bf16((N, d_model), seed + 1)
    W_K, W_V = _bf16((d_model, d_out), seed + 2, 0.05), _bf16((d_model, d_out), seed + 3, 0.05)
    W_Q, W_O = _bf16((E, d_model, d_out), seed + 4, 0.05), _bf16((E, d_out, d_model), seed + 5, 0.05)
    logits = torch.randn(N, E, generator=torch.Generator().manual_seed(seed + 6), dtype=torch.float32)
    dO = _bf16((N, d_model), seed + 7)
    return dict(X=X, W_K=W_K, W_V=W_V, W_Q=W_Q, W_O=W_O, logits=logits, dO=dO)


def _run_layer(smoe, c, B, T, E, k, h, dO=None):
    dev = lambda n: c[n].cuda()
    ei, gates = smoe.topk_gate(c["logits"].cuda(), k)
    r = smoe.route(ei, E)
    O, buf = smoe.momha_fwd(dev("X"), dev("W_K"), dev("W_V"), dev("W_Q"), dev("W_O"), r, k, gates, B, T, h, 128)
    grads = smoe.momha_bwd((c["dO"] if dO is None else dO).cuda(), dev("X"), dev("W_K"), dev("W_V"), dev("W_Q"),
                           dev("W_O"), r, k, gates, B, T, h, 128, buf)
    torch.cuda.synchronize()
    return ei.cpu().numpy(), gates.cpu().numpy().astype(np.float64), O, buf, grads   # the gates are only compared, never fed to the oracle


LAYER_SHAPES = [(2, 40, 64, 4, 2, 1), (2, 96, 256, 8, 4, 2), (1, 150, 128, 3, 3, 1)]


@pytest.mark.parametrize("B,T,d_model,E,k,h", LAYER_SHAPES)
def test_momha_layer_forward_and_backward(smoe, B, T, d_model, E, k, h):
    """Alg. 4 end to end against the oracle (routing taken from the GPU's own bit-exact top-k)."""
    _log(f"momha B={B} T={T} d_model={d_model} E={E} k={k} h={h}")
    c = _layer_case(10 * T + E, B, T, d_model, E, k, h)
    ei, g, O, buf, grads = _run_layer(smoe, c, B, T, E, k, h)
    oei, og = oracle.topk_gate(c["logits"].numpy(), k)
    assert np.array_equal(ei, oei)
    assert np.abs(g - og).max() <= 1e-6
    g = oracle_gates_f32(og)
    args = [si.as_f64(c[n]) for n in ("X", "W_K", "W_V", "W_Q", "W_O")]
    ref = oracle.momha_fwd(*args, oei, g, B, T, h, 128)
    gref = oracle.momha_bwd(si.as_f64(c["dO"]), *args, oei, g, B, T, h, 128)
    tol = TOL[torch.bfloat16]
    f64 = lambda t: t.float().cpu().numpy().astype(np.float64)
    for name, got, want in (("O", O, ref["O"]), ("K", buf.K, ref["K"]), ("V", buf.V, ref["V"]), ("Q", buf.Q, ref["Q"]),
                            ("Ohat", buf.Ohat, ref["Ohat"]), ("Yhat", buf.Yhat, ref["Yhat"])):
        err = _rel(f64(got), want)
        _log(f"  {name} rel err {err:.2e}")
        assert err <= tol, name
    for name, got in zip(("dX", "dW_K", "dW_V", "dW_Q", "dW_O", "dgates"), grads):
        err = _rel(f64(got), gref[name])
        _log(f"  {name} rel err {err:.2e}")
        assert err <= tol, name


def test_momha_layer_C5_size_prefix_subproblem(smoe):
    """Alg. 4 at the full C5 launch shape (2 x 4096 positions, d_model 2048, E 16, k 4, 4 heads of 128).
    Causality makes the first P positions of every sequence a closed sub-problem: their outputs do not
    depend on later positions, and with an upstream gradient that is zero after position P every
    gradient equals the sub-problem's.  The oracle runs that sub-problem whole."""
    B, T, d_model, E, k, h, P = 2, 4096, 2048, 16, 4, 4, 96
    c = _layer_case(77, B, T, d_model, E, k, h)
    keep = (torch.arange(B * T) % T) < P
    dO = c["dO"].clone()
    dO[~keep] = 0
    ei, g, O, buf, grads = _run_layer(smoe, c, B, T, E, k, h, dO=dO)
    _log("  GPU pass done")
    oei, og = oracle.topk_gate(c["logits"].numpy(), k)
    assert np.array_equal(ei, oei)
    assert np.abs(g - og).max() <= 1e-6
    g = oracle_gates_f32(og)
    sel = keep.numpy()
    args = [si.as_f64(c["X"])[sel]] + [si.as_f64(c[n]) for n in ("W_K", "W_V", "W_Q", "W_O")]
    ref = oracle.momha_fwd(*args, oei[sel], g[sel], B, P, h, 128)
    _log("  oracle forward done")
    gref = oracle.momha_bwd(si.as_f64(dO)[sel], *args, oei[sel], g[sel], B, P, h, 128)
    _log("  oracle backward done")
    tol = TOL[torch.bfloat16]
    f64 = lambda t: t.float().cpu().numpy().astype(np.float64)
    assert _rel(f64(O)[sel], ref["O"]) <= tol
    dX, dW_K, dW_V, dW_Q, dW_O, dg = grads
    assert np.abs(f64(dX)[~sel]).max() == 0 and np.abs(f64(dg)[~sel]).max() == 0
    for name, got, want in (("dX", f64(dX)[sel], gref["dX"]), ("dgates", f64(dg)[sel], gref["dgates"]),
                            ("dW_K", f64(dW_K), gref["dW_K"]), ("dW_V", f64(dW_V), gref["dW_V"]),
                            ("dW_Q", f64(dW_Q), gref["dW_Q"]), ("dW_O", f64(dW_O), gref["dW_O"])):
        err = _rel(got, want)
        _log(f"  {name} rel err {err:.2e}")
        assert err <= tol, name


def test_attention_C5_size_sampled_heads(smoe):
    """Attention forward and backward at C5's shape, checked on sampled (sequence, slot, head) triples: one
    slot's output and dQ involve only its own head's keys; dK/dV are checked with the upstream gradient
    restricted to that slot so that they, too, come from a single triple."""
    B, T, G, h = 2, 4096, 4, 4
    Q, K, V = _bf16((B, T, G, h, 128), 21), _bf16((B, T, h, 128), 22), _bf16((B, T, h, 128), 23)
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    O, L = smoe.attention_fwd(Qd, Kd, Vd)
    tol = TOL[torch.bfloat16]
    for b, g, hh in ((0, 0, 0), (1, 3, 2), (0, 2, 3)):
        _log(f"  triple {(b, g, hh)}")
        q1, k1, v1 = si.as_f64(Q[b:b + 1, :, g:g + 1, hh:hh + 1]), si.as_f64(K[b:b + 1, :, hh:hh + 1]), si.as_f64(V[b:b + 1, :, hh:hh + 1])
        Oref, Lref = oracle.attention_fwd(q1, k1, v1)
        assert _rel(O[b, :, g, hh].float().cpu().numpy().astype(np.float64), Oref[0, :, 0, 0]) <= tol
        assert np.abs(L[b, :, g, hh].cpu().numpy() - Lref[0, :, 0, 0]).max() <= 2e-2
        dO = torch.zeros_like(Q)
        dO[b, :, g, hh] = _bf16((T, 128), 30 + g)
        dQ, dK, dV = smoe.attention_bwd(dO.cuda(), Qd, Kd, Vd, O, L)
        rq, rk, rv = oracle.attention_bwd(si.as_f64(dO[b:b + 1, :, g:g + 1, hh:hh + 1]), q1, k1, v1)
        assert _rel(dQ[b, :, g, hh].float().cpu().numpy().astype(np.float64), rq[0, :, 0, 0]) <= tol
        assert _rel(dK[b, :, hh].float().cpu().numpy().astype(np.float64), rk[0, :, 0]) <= tol
        assert _rel(dV[b, :, hh].float().cpu().numpy().astype(np.float64), rv[0, :, 0]) <= tol
        other = dK.clone()
        other[b, :, hh] = 0
        assert other.abs().max().item() == 0          # no other head or sequence received a gradient


def test_attention_error_codes(smoe):
    import ctypes
    lib, ctx = smoe.lib, smoe.ctx()
    B, T, G, h = 1, 8, 2, 1
    Q = torch.zeros(B, T, G, h, 128, dtype=torch.bfloat16, device="cuda")
    K = torch.zeros(B, T, h, 128, dtype=torch.bfloat16, device="cuda")
    L = torch.zeros(B, T, G, h, dtype=torch.float32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    # head widths other than 128 and fp32 are valid requests this build has no kernel for
    assert lib.smoe_attention_fwd(ctx, None, smoe.BF16, p(Q), p(K), p(K), B, T, G, h, 64, p(Q), p(L)) == -2
    assert lib.smoe_attention_fwd(ctx, None, smoe.F32, p(Q), p(K), p(K), B, T, G, h, 128, p(Q), p(L)) == -2
    assert lib.smoe_attention_fwd(ctx, None, smoe.BF16, None, p(K), p(K), B, T, G, h, 128, p(Q), p(L)) == -1
    assert lib.smoe_attention_fwd(ctx, None, smoe.BF16, p(Q), p(K), p(K), B, 0, G, h, 128, p(Q), p(L)) == -1
    need = lib.smoe_attention_bwd_workspace_bytes(B, T, G, h)
    assert need >= B * T * G * h * 4
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    rc = lib.smoe_attention_bwd(ctx, None, smoe.BF16, p(Q), p(Q), p(K), p(K), p(Q), p(L), B, T, G, h, 128, p(Q), p(K), p(K),
                                p(ws), 16)
    assert rc == -3            # workspace too small
    with pytest.raises(smoe.SmoeError):
        smoe.attention_fwd(torch.zeros(1, 4, 1, 1, 64, dtype=torch.bfloat16, device="cuda"),
                           torch.zeros(1, 4, 1, 64, dtype=torch.bfloat16, device="cuda"),
                           torch.zeros(1, 4, 1, 64, dtype=torch.bfloat16, device="cuda"))


def test_attention_is_deterministic(smoe):
    B, T, G, h = 2, 200, 3, 2
    Q, K, V, dO = (_bf16(s, i).cuda() for i, s in enumerate([(B, T, G, h, 128), (B, T, h, 128), (B, T, h, 128), (B, T, G, h, 128)]))
    O1, L1 = smoe.attention_fwd(Q, K, V)
    g1 = smoe.attention_bwd(dO, Q, K, V, O1, L1)
    O2, L2 = smoe.attention_fwd(Q, K, V)
    g2 = smoe.attention_bwd(dO, Q, K, V, O2, L2)
    assert torch.equal(O1, O2) and torch.equal(L1, L2)
    for a, b in zip(g1, g2):
        assert torch.equal(a, b)


def _raw_layer_backward(m, c, r, k, gates, B, T, h, buf, dO, X, dX, dW):
    """smoe_momha_bwd with the caller's own dX and dW tensors; returns the status."""
    d_model = c["X"].shape[1]
    nb = m.lib.smoe_momha_bwd_workspace_bytes(B, T, k, d_model, h, 128)
    ws = m._ws(nb, "cuda")
    rc = r.c()
    weights = [c[n].cuda() for n in ("W_K", "W_V", "W_Q", "W_O")]
    dg = torch.full_like(gates, 7.0)
    status = m.lib.smoe_momha_bwd(m.ctx(), m._stream(), m.BF16, m._p(dO), m._p(X), B, T, d_model, h, 128, *(m._p(w) for w in weights),
                                  ctypes.byref(rc), k, m._p(gates), m._p(buf.K), m._p(buf.V), m._p(buf.Q), m._p(buf.Ohat),
                                  m._p(buf.LSE), m._p(buf.Yhat), m._p(dX), *(m._p(w) for w in dW), m._p(dg), m._p(ws), nb)
    torch.cuda.synchronize()
    return status, dg


@pytest.mark.parametrize("k", [1, 2])
def test_momha_backward_pointers_off_16_byte_lines(smoe, k):
    """dX may lie anywhere its elements can: the call writes it like an aligned one.  An X the sorted copies cannot read is
    refused before anything is written."""
    B, T, d_model, E, h = 1, 70, 64, 4, 1
    _log(f"momha backward off 16-byte lines k={k}")
    c = _layer_case(5, B, T, d_model, E, k, h)
    ei, gates = smoe.topk_gate(c["logits"].cuda(), k)
    r = smoe.route(ei, E)
    X, dO = c["X"].cuda(), c["dO"].cuda()
    args = [X] + [c[n].cuda() for n in ("W_K", "W_V", "W_Q", "W_O")]
    _, buf = smoe.momha_fwd(*args, r, k, gates, B, T, h, 128)
    want = smoe.momha_bwd(dO, *args, r, k, gates, B, T, h, 128, buf)
    off = lambda t: torch.full((t.numel() + 8,), 7.0, dtype=t.dtype, device="cuda")[4:4 + t.numel()].view(t.shape)
    empty = lambda: [torch.full_like(t, 7.0) for t in want[1:5]]
    dX, dW = off(X), empty()
    assert dX.data_ptr() % 16 == 8
    status, dg = _raw_layer_backward(smoe, c, r, k, gates, B, T, h, buf, dO, X, dX, dW)
    assert status == 0
    for got, ref in zip([*dW, dg], want[1:]):
        assert torch.equal(got, ref)
    # the three parts of dX may be added in two steps here and in one there: one rounding to 8 bits more
    assert float((dX.float() - want[0].float()).abs().max()) <= 2 ** -7 * float(want[0].float().abs().max())
    X_off = off(X)
    X_off.copy_(X)
    dX, dW = torch.full_like(X, 7.0), empty()
    status, dg = _raw_layer_backward(smoe, c, r, k, gates, B, T, h, buf, dO, X_off, dX, dW)
    assert status == -2
    assert all(bool((t == 7.0).all()) for t in [dX, dg, *dW]), "a refused call wrote to an output"
