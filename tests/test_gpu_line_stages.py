"""GPU parity of the persistent kernels' stages of 64 contraction elements where they can go wrong: contractions of two to five
stages that end on, one chunk (8 elements) behind and one chunk before the end of a stage, with enough tiles per block for the ring
of order indices and open tiles to come round more than once (two stages per tile is the least it is laid out for), and segments
that leave rows of a tile empty (these read zeros).  Every row is compared with the oracle on sampled columns."""
import numpy as np
import pytest
import torch

import oracle
import smoe_inputs as si
from helpers import assert_close, oracle_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[3, 4], ids=["tiles128", "tiles256"])
def smoe(request):
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.set_kernel_mode(request.param)
    yield m
    m.set_kernel_mode(0)


# K: the contraction of the forward product (d_in); N: that of the input gradient (d_out).  At least five tiles of 256 rows per block
# in one direction each: 2 * T rows make 94 tiles of 256 rows or more.
@pytest.mark.parametrize("K,N", [(72, 3848), (128, 3848), (136, 3848), (184, 3848), (192, 3848), (264, 3848), (3848, 72), (3848, 128), (3848, 136), (3848, 320)])
def test_short_contractions_over_several_rounds(smoe, K, N):
    T, E, k = 12000, 6, 2
    assert (-(-T * k // 256)) * (-(-max(K, N) // 256)) >= 5 * 256
    c = si.plinear_case(T, K, N, E, k, "bf16", seed=77)
    ei, _, se, o, off = oracle_routing(c["logits"], k, E)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    X, W, dY = c["X"].cuda(), c["W"].cuda(), c["dY_Tk"].cuda()
    print("stages", K, N, np.diff(off).tolist(), flush=True)
    X64, W64, dY64 = si.as_f64(c["X"]), si.as_f64(c["W"]), si.as_f64(c["dY_Tk"])
    pick = lambda n: np.unique(np.concatenate([np.arange(0, n, 241), [max(0, n - 1)]]))
    cols, rows = pick(N), pick(K)
    Y, _ = smoe.plinear_fwd(X, W, r, k, None, False, False)                  # gathered rows, scattered output
    Y_ref, _ = oracle.plinear_fwd(X64, W64[:, :, cols], se, o, k, None, False, False)
    assert_close(Y[:, torch.from_numpy(cols).cuda()], Y_ref, torch.bfloat16, "Y")
    dX, _, _ = smoe.plinear_bwd(dY, X, W, None, r, k, None, False, True)     # sorted rows, W^T, scattered output
    dX_ref, _, _ = oracle.plinear_bwd(dY64, X64[:, rows], W64[:, rows, :], se, o, k, None, False, True)
    assert_close(dX[:, torch.from_numpy(rows).cuda()], dX_ref, torch.bfloat16, "dX")
    for name, t in (("Y", Y), ("dX", dX)):
        assert bool(torch.isfinite(t.float()).all()), f"{name} holds entries no kernel wrote"
