"""The fp32 matrix-core kernels where they can go wrong: contractions and widths around their 32- and 64-element tiles, the
paired gate / up tile of SwiGLU partly empty, segments at the 64-row tile's edges, empty experts, gathered and weighted rows
(no sorted copies are made).  Against the fp64 oracle at 1e-5 of the tensor's (and of each row's) largest entry: sums of up
to a few hundred fp32 terms."""
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


@pytest.mark.parametrize("act", [si.ACT_NONE, si.ACT_GELU, si.ACT_SWIGLU])
@pytest.mark.parametrize("T,d_model,d_expert,E,k,masked", [(1, 4, 4, 1, 1, 0), (64, 32, 64, 1, 1, 0), (130, 28, 36, 2, 2, 0), (200, 36, 28, 3, 1, 0),
                                                           (257, 68, 100, 5, 3, 2), (193, 128, 132, 70, 4, 10), (40, 36, 32, 11, 9, 0)])
def test_mlp_every_row(smoe, T, d_model, d_expert, E, k, masked, act):
    cfg = si.custom("f32-edges", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=act, dtype="f32", masked_experts=masked)
    case = si.mlp_case(cfg, 71)
    ei, g, se, o, off = oracle_routing(case["logits"], k, E)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    print("f32 mlp", T, d_model, d_expert, E, k, act, flush=True)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    Y, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, act)
    Yi, _ = smoe.mlp_fwd(X, W1, W2, r, k, gg, act, training=False)
    assert torch.equal(Y, Yi)                    # the pre-activation need not be kept
    grads = smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf)
    g64 = oracle_gates_f32(g)
    args = [si.as_f64(case[n]) for n in ("X", "W1", "W2")]
    ref = oracle.mlp_fwd(*args, ei, g64, act)
    gref = oracle.mlp_bwd(si.as_f64(case["dY"]), *args, ei, g64, act)
    for got, want, nm in zip((Y,) + tuple(grads), (ref["Y"], gref["dX"], gref["dW1"], gref["dW2"], gref["dgates"]), ("Y", "dX", "dW1", "dW2", "dgates")):
        assert_close(got, want, torch.float32, nm)
