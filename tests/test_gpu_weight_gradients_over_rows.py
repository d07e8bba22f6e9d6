"""Both weight gradients of the MLP in one launch with outputs that lie over its inputs: no operand is read through the order indices then,
sorted copies of X and dY stand in, and the gradients are those of a call with outputs of their own, bit for bit.  Only where the hidden
rows carry the routing weights in place of the copy of dY (SwiGLU, no wider than the model) is the rounding of dW2 another one, and the
oracle decides."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing
from test_gpu_weight_gradients_together import _taken

pytestmark = pytest.mark.gpu


def _over(mem, rows):
    place = mem.view(-1).view(rows.dtype)[:rows.numel()].view_as(rows)
    place.copy_(rows)
    return place


@pytest.mark.parametrize("T,d_model,d_expert,E,k,act", [
    (140, 1032, 1416, 9, 1, si.ACT_SWIGLU),       # weighted copy of dY, gathered copies
    (70, 1032, 1416, 9, 2, si.ACT_SWIGLU),
    (70, 1288, 1032, 9, 2, si.ACT_GELU),          # weighted hidden rows beside a plain copy of dY
    (70, 1288, 1032, 9, 2, si.ACT_SWIGLU),
])
def test_outputs_over_inputs(T, d_model, d_expert, E, k, act):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    assert _taken(smoe, d_model, d_expert, E, act) and T * k * d_model * 2 <= 64 << 20
    cfg = si.custom("together-over", T=T, d_model=d_model, d_expert=d_expert, E=E, k=k, act=act, dtype="bf16", masked_experts=1)
    case = si.mlp_case(cfg, 96)
    ei, g, _, _, _ = oracle_routing(case["logits"], k, E)
    gi, gg = smoe.topk_gate(case["logits"].cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    r = smoe.route(gi, E)
    X, W1, W2, dY = (case[n].cuda() for n in ("X", "W1", "W2", "dY"))
    _, buf = smoe.mlp_fwd(X, W1, W2, r, k, gg, act)
    assert buf.Yhat is None          # the persistent kernels take these widths
    names = ("dX", "dW1", "dW2", "dgates")
    want = [t.clone() for t in smoe.mlp_bwd(dY, X, W1, W2, r, k, gg, act, buf)]
    ref = oracle.mlp_bwd(si.as_f64(case["dY"]), *[si.as_f64(case[n]) for n in ("X", "W1", "W2")], ei, oracle_gates_f32(g), act)
    for t, n in zip(want, names):
        assert_close(t, ref[n], torch.bfloat16, n)
    bits = not (act == si.ACT_SWIGLU and d_expert <= d_model)
    for out, rows in (("dW1", "X"), ("dW1", "dY"), ("dW2", "X"), ("dW2", "dY"), ("dgates", "dY")):
        print("outputs over inputs", T, d_model, d_expert, k, act, out, "over", rows, flush=True)
        given = {"X": X, "dY": dY}
        own = getattr(buf, out)
        if out == "dgates":              # the small one lies in the rows
            mem = given[rows].clone()
            given[rows] = mem
            setattr(buf, out, mem.view(-1).view(torch.float32)[:own.numel()].view_as(own))
        else:
            mem = torch.empty_like(own)
            given[rows] = _over(mem, given[rows])
            setattr(buf, out, mem)
        got = smoe.mlp_bwd(given["dY"], given["X"], W1, W2, r, k, gg, act, buf)
        for t, w, n in zip(got, want, names):
            if bits or n != "dW2":
                assert torch.equal(t, w), f"{n} ({out} over {rows})"
            else:
                assert_close(t, ref[n], torch.bfloat16, f"{n} ({out} over {rows})")
        setattr(buf, out, own)
