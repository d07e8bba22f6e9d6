"""ParallelLinear backward whose two sorted copies and row dots are one launch (rows shared by k > 1 slots, copies of 24 Mi elements
or more): widths whose rows take one, three and four wavefronts, k with and without a loop of its own.  Every row of dX and dW at
sampled input features, the routing-weight gradient of sampled tokens, against the oracle; and bit for bit the weight gradient of
the same rows copied one after the other."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_gates_f32, oracle_routing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_in,d_out,E,k", [(2010, 1176, 1960, 5, 4), (940, 2048, 1000, 12, 9), (6300, 504, 1544, 4, 2)])
def test_copies_and_row_dots(T, d_in, d_out, E, k):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    assert T * k * (d_in + d_out) >= 24 << 20        # the launch under test is taken
    c = si.plinear_case(T, d_in, d_out, E, k, "bf16", seed=101)
    ei, g, se, o, off = oracle_routing(c["logits"], k, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    gg = torch.from_numpy(g.astype(np.float32)).cuda()
    print("spread", T, d_in, d_out, E, k, np.diff(off).tolist(), flush=True)
    X, W, dY = c["X"].cuda(), c["W"].cuda(), c["dY_T"].cuda()
    _, Yhat = smoe.plinear_fwd(X, W, r, k, gg)
    dX, dW, dg = smoe.plinear_bwd(dY, X, W, Yhat, r, k, gg)
    # one at a time: the sorted copies as launches of their own, and the weight gradient of grouped rows
    dW1 = smoe.plinear_bwd(smoe.group(dY, r, k, gg), smoe.group(X, r, k), W, None, r, 1, None, True, True)[1]
    assert torch.equal(dW, dW1)
    rng = np.random.default_rng(3)
    cols = np.sort(rng.choice(d_in, 12, replace=False))
    X64, W64, dY64, g64 = si.as_f64(c["X"]), si.as_f64(c["W"]), si.as_f64(c["dY_T"]), oracle_gates_f32(g)
    dX_ref, dW_ref, _ = oracle.plinear_bwd(dY64, X64[:, cols], W64[:, cols, :], se, o, k, g64, False, False)
    ct = torch.from_numpy(cols).cuda()
    assert_close(dX[:, ct], dX_ref, torch.bfloat16, "dX")
    assert_close(dW[:, ct, :], dW_ref, torch.bfloat16, "dW")
    S = np.sort(rng.choice(T, 96, replace=False))
    se_s, o_s, _ = oracle.route(ei[S], E)
    _, _, dp_ref = oracle.plinear_bwd(dY64[S], X64[S], W64, se_s, o_s, k, g64[S], False, False)
    assert_close(dg[torch.from_numpy(S).cuda()], dp_ref, torch.bfloat16, "dgates")
