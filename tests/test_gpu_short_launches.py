"""Forward products on 128 x 256 tiles, with two stages of operands in flight (contractions of up to four stages of 64, or one round of tiles
with up to eight stages or rows of W at a stride of whole kilobytes) and with three: the same bits as on the 256 x 256 tiles, whose sums run in the same order.  Contractions of two stages and a few
elements up to several stages and a remainder, widths that end inside a tile, experts without rows, with one row, with a whole tile and a
row; one round, several; W read through the caches and, where a call's weights exceed them, past them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
GRID, ROWS, COLS = 256, 128, 256


def _routed(smoe, loads, k, seed):
    rng = np.random.default_rng(seed)
    slots = rng.permutation(np.repeat(np.arange(len(loads), dtype=np.int32), loads))
    return smoe.route(torch.from_numpy(slots.reshape(-1, k)).cuda(), len(loads)), len(slots)


def _compare(smoe, loads, k, d_in, width, seed, swiglu=True):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    r, Tk = _routed(smoe, loads, k, seed)
    X, W = normal(Tk // k, d_in), normal(len(loads), d_in, width).mul_(d_in ** -0.5)
    got = {}
    for mode in (3, 4):
        print("short launches", Tk, len(loads), k, d_in, width, "mode", mode, flush=True)
        smoe.set_kernel_mode(mode)
        try:
            out = [smoe.plinear_fwd(X, W, r, k, None, False, g)[1] for g in (False, True)]
            if swiglu:
                out += list(smoe.plinear_act_fwd(X, W, r, k, smoe.ACT_SWIGLU)) + [smoe.plinear_act_fwd(X, W, r, k, smoe.ACT_SWIGLU, keep_hpre=False)[0]]
        finally:
            smoe.set_kernel_mode(0)
        got[mode] = out
    for a, b in zip(got[3], got[4]):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert all(bool(torch.isfinite(t.float()).all()) for t in got[3])
    # one expert's rows against the product in fp32: the sums of 16-bit products, rounded once
    e = int(np.argmax(loads))
    lo = int(np.sum(loads[:e]))
    rows = torch.div(r.sorted_scattered_idxs[lo:lo + loads[e]].long(), k, rounding_mode="floor")
    want = X[rows].double() @ W[e].double()
    assert (got[3][1][lo:lo + loads[e]].double() - want).abs().max() <= 2.0 ** -8 * want.abs().max()


LOADS = [0, 1, 129, 64, 127, 128, 200, 3, 257, 31]


@pytest.mark.parametrize("d_in,width", [(d, w) for d in (72, 128, 192, 200, 256, 264, 456, 512) for w in (272, 1040)] +
                         [(520, 1040), (520, 1024), (776, 512), (1032, 1536)])
def test_one_round(d_in, width):
    import paper_2403_08245_amd as smoe
    assert torch.cuda.is_available(), "these tests need the MI355X"
    assert sum(-(-n // ROWS) for n in LOADS) * -(-width // COLS) <= GRID
    _compare(smoe, LOADS, 2, d_in, width, d_in)


@pytest.mark.parametrize("d_in", [72, 200, 256, 264, 456])
def test_several_rounds(d_in):
    import paper_2403_08245_amd as smoe
    width, loads = 2576, [n * 3 for n in LOADS]
    assert sum(-(-n // ROWS) for n in loads) * -(-width // COLS) > GRID and sum(loads) // ROWS * (width // COLS) > GRID * 3 // 4
    _compare(smoe, loads * 2, 4, d_in, width, d_in + 1)


@pytest.mark.parametrize("E,d_in,width,rows", [(20, 2056, 3344, 60), (40, 1160, 3088, 60)])   # 260 and 520 tiles at 13 per expert
def test_weights_past_the_caches(E, d_in, width, rows):
    import paper_2403_08245_amd as smoe
    loads = [rows] * E
    loads[0], loads[1], loads[2] = 0, 130, 2 * rows - 10
    assert E * d_in * width * 2 > 256 << 20 and sum(loads) <= ROWS * E
    _compare(smoe, loads, 1, d_in, width, E)


@pytest.mark.parametrize("width", [2048, 2064])
def test_weights_past_the_caches_in_one_round(width):
    import paper_2403_08245_amd as smoe
    loads = [0, 130] + [60] * 14 + [50]
    assert 17 * 4104 * width * 2 > 256 << 20 and 17 * -(-width // COLS) <= GRID and sum(loads) <= ROWS * 17
    _compare(smoe, loads, 1, 4104, width, 8)


@pytest.mark.parametrize("d_expert", [4096, 4104])
def test_cut_contraction(d_expert):
    """The second product of an MLP, whose few tiles are cut along the contraction, from the hidden rows that the pass kept."""
    import paper_2403_08245_amd as smoe
    T, d_model, E, k = 480, 1024, 8, 2
    gen = torch.Generator(device="cuda").manual_seed(d_expert)
    normal = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    X, W1, W2 = normal(T, d_model), normal(E, d_model, 2 * d_expert).mul_(d_model ** -0.5), normal(E, d_expert, d_model).mul_(d_expert ** -0.5)
    ei, g = smoe.topk_gate(torch.empty(T, E, device="cuda").normal_(generator=gen), k)
    r = smoe.route(ei, E)
    assert 32 * E < T * k <= ROWS * E and E * d_model // COLS * 4 <= GRID and d_model % 512 == 0
    print("cut contraction", d_expert, flush=True)
    smoe.set_kernel_mode(3)
    try:
        Y, buf = smoe.mlp_fwd(X, W1, W2, r, k, g, smoe.ACT_SWIGLU)
    finally:
        smoe.set_kernel_mode(0)
    off, o = r.expert_offsets.tolist(), r.sorted_scattered_idxs.long()
    want = torch.zeros(T, d_model, dtype=torch.float64, device="cuda")
    for e in range(E):
        s = o[off[e]:off[e + 1]]
        want.index_add_(0, s // k, g.view(-1)[s].double()[:, None] * (buf.H[off[e]:off[e + 1]].double() @ W2[e].double()))
    # every slot's row is rounded once to 8 significant bits, and their weighted sum once more
    assert (Y.double() - want).abs().max() <= 2.0 ** -7 * want.abs().max()
