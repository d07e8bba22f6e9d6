"""Routing at the sizes where its dispatch changes: wavefront, block and chunk edges of the one-launch sort, the first sizes
of the two- and three-launch ones, expert counts on both sides of the replicated histograms, one popular expert, and top-k
at the limits of the k-rounds selection.  Integer results are bit-exact against the oracle; gates at 1e-6."""
import numpy as np
import pytest
import torch

import oracle
from helpers import oracle_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2403_08245_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return m


@pytest.mark.parametrize("Tk,E", [(1, 1), (63, 5), (64, 64), (65, 3), (255, 64), (256, 64), (257, 64), (1024, 8), (1025, 256), (2047, 257),
                                  (32768, 64), (32769, 64), (40000, 2), (33000, 992), (33000, 993), (3000, 8192), (3000, 8193), (70000, 600),
                                  (0, 16384), (1, 16384), (200, 8193), (1000, 16384), (3000, 16384), (40000, 16384)])
@pytest.mark.parametrize("popular", [False, True])
def test_stable_sort(smoe, Tk, E, popular):
    rng = np.random.default_rng(Tk * 7 + E)
    ei = rng.integers(0, E, size=(Tk, 1)).astype(np.int32)
    if popular and Tk:
        ei[rng.random(Tk) < 0.9] = E // 2
    print("sort", Tk, E, popular, flush=True)
    r = smoe.route(torch.from_numpy(ei).cuda(), E)
    e = ei[:, 0].astype(np.int64)
    o = np.argsort(e, kind="stable")
    assert np.array_equal(r.sorted_scattered_idxs.cpu().numpy(), o)
    assert np.array_equal(r.sorted_expert_idxs.cpu().numpy(), e[o])
    assert np.array_equal(r.expert_offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(e, minlength=E))]))


@pytest.mark.parametrize("Tk,E", [(1, 5), (64, 8192), (300, 8193), (1024, 16384)])
def test_one_chunk_leaves_the_scratch_alone(smoe, Tk, E):
    """Up to 1024 slots the counts never leave LDS, whatever the number of experts: calls that share a scratch do not meet in it
    (smoe_route_noalloc keeps one per device)."""
    print("scratch", Tk, E, flush=True)
    ei = torch.from_numpy(np.random.default_rng(Tk).integers(0, E, size=(Tk, 1)).astype(np.int32)).cuda()
    want = smoe.route(ei, E)
    ws = torch.full((smoe.lib.smoe_route_workspace_bytes(Tk, 1, E),), 0x5A, dtype=torch.uint8, device="cuda")
    se, so = torch.empty(Tk, dtype=torch.int32, device="cuda"), torch.empty(Tk, dtype=torch.int32, device="cuda")
    off = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    assert smoe.lib.smoe_route(smoe.ctx(), smoe._stream(), smoe._p(ei), Tk, 1, E, smoe._p(se), smoe._p(so), smoe._p(off), smoe._p(ws), ws.numel()) == 0
    assert torch.equal(so, want.sorted_scattered_idxs) and torch.equal(off, want.expert_offsets)
    assert bool((ws == 0x5A).all())


@pytest.mark.parametrize("E,k", [(24, 24), (64, 24), (64, 25), (65, 64), (128, 64), (129, 65), (256, 64), (257, 9), (1024, 64), (1025, 3)])
def test_topk_limits(smoe, E, k):
    gen = torch.Generator().manual_seed(E + k)
    logits = torch.randint(-40, 40, (301, E), generator=gen).to(torch.float32) / 8       # ties on purpose
    logits[torch.rand(301, E, generator=gen) < 0.05] = -float("inf")
    logits[torch.rand(301, E, generator=gen) < 0.05] = float("nan")
    logits[5] = -0.0
    logits[5, ::2] = 0.0                                                                  # equal to -0.0: lower id first
    print("topk", E, k, flush=True)
    ei, g, _, _, _ = oracle_routing(logits, k, E)
    gi, gg = smoe.topk_gate(logits.cuda(), k)
    assert np.array_equal(gi.cpu().numpy(), ei)
    assert np.abs(gg.cpu().numpy().astype(np.float64) - g).max() <= 1e-6
