"""Kernels whose workgroups exchange a step's values through the L2 of one XCD.  A single sequence: lengths around the chunks of
steps whose reserve values pass through LDS together, one and more layers; the same bits with stores that write through to memory
(LSTM_FULL_FENCES), which is what a layer spread over XCDs uses."""
import pytest

from paper_1604_01946_amd.inputs import Config
from parity import recurrence_kernels
from test_gpu_in_place import lstm as lstm_pass, same
from test_gpu_in_place import test_cells as test_states_in_place_of_other_cells  # noqa: F401  (there without these kernels)
from test_gpu_parity import BWD, FWD, run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu


def cfg(L, T, B, I, H):
    return Config("near", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)


@pytest.mark.parametrize("H", [128, 256, 512])
@pytest.mark.parametrize("L,T,I", [(1, 7, 0), (1, 8, 24), (2, 8, 0), (3, 9, 24), (2, 16, 24), (2, 17, 0), (8, 10, 0)])
def test_single_sequence(H, L, T, I, knobs):
    knobs(LSTM_FULL_FENCES="1")
    slow, _ = run_case(cfg(L, T, 1, I or H, H), 21, 6)
    knobs(LSTM_FULL_FENCES=None)
    fast, _ = run_case(cfg(L, T, 1, I or H, H), 21, 6)
    for k in FWD + BWD:
        assert (getattr(slow, k) == getattr(fast, k)).all(), k


# The kernels with step counters, which run where these two settings ask for them or the device has fewer CUs: a single sequence, a batch of
# one slice, slices of 16 rows side by side; the other cells on the alternating kernels.
NARROW = [(2, 5, 1, 0, 192), (2, 9, 1, 24, 256), (2, 5, 16, 0, 128), (1, 4, 17, 24, 256), (2, 3, 64, 0, 256), (1, 9, 64, 0, 512), (3, 4, 33, 24, 192)]


@pytest.mark.parametrize("L,T,B,I,H", NARROW)
def test_lstm_on_the_kernels_with_step_counters(L, T, B, I, H, knobs):
    c = cfg(L, T, B, I or H, H)
    if B == 1:
        knobs(LSTM_TINY="0")
        assert recurrence_kernels(lambda: run_case(c, 25, 6)) == ("pers_fwd_kernel", "pers_bwd_kernel")
        knobs(LSTM_TINY=None)
        assert recurrence_kernels(lambda: run_case(c, 25, 6)) == ("pers_fwd_tiny_kernel", "pers_bwd_tiny_kernel")
    else:
        knobs(LSTM_NEAR="0")
        assert recurrence_kernels(lambda: run_case(c, 25, 6)) == ("pers_fwd_kernel", "pers_bwd_kernel")
        knobs(LSTM_NEAR=None)
        assert recurrence_kernels(lambda: run_case(c, 25, 6)) == ("pers_fwd_near_kernel", "pers_bwd_near_kernel")


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("L,T,B,I,H", [(2, 5, 1, 0, 192), (2, 5, 16, 0, 128), (1, 4, 17, 24, 256), (2, 3, 32, 0, 512)])
def test_other_cells_on_the_alternating_kernels(cell, L, T, B, I, H, knobs):
    call = lambda: run_cell(cell, L, T, B, I or H, H, seed=4)  # noqa: E731
    assert recurrence_kernels(call) == ("pers_fwd_near_kernel", "pers_bwd_near_kernel")
    knobs(LSTM_NEAR="0")
    assert recurrence_kernels(call)[1] == "pers_bwd_pp_kernel"


# Slices of 16 rows: 8 and 16 (single gate 16 and 32) units per workgroup, groups on one XCD, two on one, on all; rows that do not
# fill a slice; one, two and three steps; every size that has instances of its own.
SLICES = [
    (1, 3, 16, 0, 128), (2, 5, 17, 40, 128), (4, 3, 64, 0, 128), (8, 2, 5, 0, 128), (3, 4, 33, 24, 192), (2, 2, 100, 0, 192),
    (1, 1, 40, 0, 256), (4, 6, 64, 0, 256), (2, 3, 2, 300, 256), (8, 3, 15, 24, 256), (3, 5, 17, 0, 320), (1, 17, 31, 0, 320),
    (2, 4, 20, 24, 384), (1, 9, 64, 0, 384), (3, 2, 16, 0, 448), (4, 5, 3, 24, 512), (1, 10, 33, 0, 512),
]


@pytest.mark.parametrize("L,T,B,I,H", SLICES)
def test_slices_lstm(L, T, B, I, H, knobs):
    knobs(LSTM_FULL_FENCES="1")
    slow, _ = run_case(cfg(L, T, B, I or H, H), 22, 6)
    knobs(LSTM_FULL_FENCES=None)
    fast, _ = run_case(cfg(L, T, B, I or H, H), 22, 6)
    for k in FWD + BWD:
        assert (getattr(slow, k) == getattr(fast, k)).all(), k


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("L,T,B,I,H", SLICES + [(2, 3, 1, 0, 256), (3, 12, 1, 24, 512), (4, 3, 300, 0, 256), (1, 9, 530, 24, 512)])
def test_slices_other_cells(cell, L, T, B, I, H):
    run_cell(cell, L, T, B, I or H, H, seed=4)


# Many slices: their bias gradients fill up to half of the area that they are left in, which holds 64 rows of 4H.  (One of 16 x 64 rows, one
# more, as many as these cells have on chip, and a padded size.)
@pytest.mark.parametrize("cell", ["tanh", "relu"])
@pytest.mark.parametrize("B,H", [(1024, 128), (1025, 128), (2048, 128), (2040, 100)])
@pytest.mark.parametrize("with_h0", [True, False])
def test_many_slices(cell, B, H, with_h0):
    run_cell(cell, 2, 2, B, 24, H, seed=4, with_h0=with_h0)


def test_bias_gradients_of_many_slices_stay_in_their_area():
    """Behind that area the workspace has [8][B][4H] floats for paths that run unfused, which these kernels leave alone: the longest
    run of words that a pass of one step does not write (the exchange area and the stand-in of the reserve together are smaller)."""
    import torch

    from paper_1604_01946_amd import binding as Bd
    from test_gpu_rnn_cells import make

    cell, L, T, B, I, H = "tanh", 2, 1, 2048, 24, 128
    c, t = Bd.RNN_CELLS[cell], {k: torch.from_numpy(v).cuda() for k, v in make(cell, L, T, B, I, H, 4).items()}
    rb, wb = Bd.rnn_reserve_bytes(c, L, T, B, I, H), Bd.rnn_workspace_bytes(c, L, T, B, I, H)
    res, ws = torch.empty(rb // 4, device="cuda"), torch.empty(wb // 4, dtype=torch.int32, device="cuda")
    y, new = torch.empty(T, B, H, device="cuda"), lambda k: torch.empty_like(t[k])
    Bd.check(Bd.rnn_forward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], t["b"], y, None, res, ws, wb), "rnn_forward")
    ws.fill_(0x7EADBEEF)
    Bd.check(Bd.rnn_backward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], res, t["dy"], t["dhT"], new("x"), new("h0"), new("W"), new("R"),
                             new("b"), ws, wb), "rnn_backward")
    written = torch.nonzero(ws != 0x7EADBEEF).flatten()
    ends = torch.cat([written.new_tensor([-1]), written, written.new_tensor([ws.numel()])])
    assert (ends.diff().max() - 1).item() >= 8 * B * 4 * H


# Sizes with one-layer kernels as well: LSTM and GRU up to 896 layer by layer, lengths on both sides of the lines between the kernels, the single
# gate with all layers in a launch, with groups of them, and in several launches; padded to these sizes.
LARGE = [(1, 1, 16, 0, 640), (2, 9, 33, 24, 640), (2, 5, 32, 0, 768), (1, 17, 17, 0, 768), (3, 8, 5, 24, 896), (1, 3, 32, 0, 896), (2, 6, 20, 0, 1024), (2, 4, 3, 40, 700)]


@pytest.mark.parametrize("L,T,B,I,H", LARGE)
def test_large_lstm(L, T, B, I, H):
    run_case(cfg(L, T, B, I or H, H), 23, 0)


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("L,T,B,I,H", LARGE + [(6, 3, 20, 0, 896), (5, 4, 3, 0, 1024), (1, 5, 100, 0, 1024), (2, 3, 130, 24, 768)])
def test_large_other_cells(cell, L, T, B, I, H):
    run_cell(cell, L, T, B, I or H, H, seed=4)


# Short passes above 512 units: both sides of the lines between these kernels and the one-layer kernels.
@pytest.mark.parametrize("cell,L,T,B,H,near", [
    ("tanh", 4, 2, 177, 846, (1, 0)), ("tanh", 6, 3, 98, 896, (0, 0)), ("tanh", 3, 3, 180, 1024, (1, 0)), ("tanh", 2, 3, 65, 1024, (1, 1)), ("tanh", 4, 14, 98, 1024, (1, 1)),
    ("relu", 7, 2, 112, 896, (0, 0)), ("lstm", 1, 2, 10, 708, (1, 0)), ("lstm", 1, 8, 20, 768, (1, 1)), ("lstm", 2, 3, 20, 768, (1, 1)), ("gru", 1, 2, 6, 734, (1, 0)),
    ("gru", 1, 12, 20, 896, (1, 0)), ("gru", 1, 3, 20, 640, (1, 1)), ("lstm", 1, 2, 20, 640, (1, 0))])
def test_short_passes_above_512_units(cell, L, T, B, H, near):
    names = recurrence_kernels(lambda: run_case(cfg(L, T, B, 24, H), 26, 0) if cell == "lstm" else run_cell(cell, L, T, B, 24, H, seed=4))
    assert (names[0] == "pers_fwd_near_kernel", names[1] == "pers_bwd_near_kernel") == tuple(map(bool, near)), names


# hT = h0, cT = c0, dh0 = dhT, dc0 = dcT: one XCD and all, one launch per layer and all layers in one, a single sequence.
@pytest.mark.parametrize("dims", [(2, 9, 1, 24, 256), (4, 3, 64, 128, 128), (3, 5, 17, 320, 320), (2, 4, 20, 24, 384), (1, 10, 33, 512, 512), (2, 9, 33, 24, 640)])
@pytest.mark.parametrize("nan", [False, True])
def test_states_in_place(dims, nan):
    got = {}
    assert recurrence_kernels(lambda: got.update(lstm_pass(dims, nan, True, 0)))[0] == ("pers_fwd_tiny_kernel" if dims[2] == 1 else "pers_fwd_near_kernel")
    same(lstm_pass(dims, nan, False, 0), got)


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("H,B", [(256, 20), (320, 5), (896, 18)])
def test_a_row_of_other_cells_that_is_not_finite_spoils_no_other(cell, H, B):
    import numpy as np
    import torch

    from paper_1604_01946_amd import binding as Bd
    from test_gpu_rnn_cells import make

    L, T, I, c, out = 2, 4, 24, Bd.RNN_CELLS[cell], []
    for spoil in (False, True):
        d = make(cell, L, T, B, I, H, 4)
        if spoil:
            d["x"][1, 2, 5], d["x"][2, 3, :], d["h0"][:, 4, 7] = np.nan, np.inf, np.nan
        t = {k: torch.from_numpy(v).cuda() for k, v in d.items()}
        rb, wb = Bd.rnn_reserve_bytes(c, L, T, B, I, H), Bd.rnn_workspace_bytes(c, L, T, B, I, H)
        res, ws = torch.empty(rb // 4, device="cuda"), torch.empty(wb // 4, device="cuda")
        y, new = torch.empty(T, B, H, device="cuda"), lambda k: torch.empty_like(t[k])
        hT, dx, dh0 = new("h0"), new("x"), new("h0")

        def call():
            Bd.check(Bd.rnn_forward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], t["b"], y, hT, res, ws, wb), "rnn_forward")
            Bd.check(Bd.rnn_backward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], res, t["dy"], t["dhT"], dx, dh0, new("W"), new("R"), new("b"), ws, wb), "rnn_backward")

        assert recurrence_kernels(call) == ("pers_fwd_near_kernel", "pers_bwd_near_kernel" if H < 896 or cell not in ("gru",) else "pers_bwdL_kernel")
        out.append((y, hT, dx, dh0))
    keep = [b for b in range(B) if b not in (2, 3, 4)]
    for a, b in zip(*out):
        # (as above: sums of a tile with one that is not finite are worked out with other instructions)
        assert (a[:, keep] - b[:, keep]).abs().max() <= 1e-5 * a.abs().max()
    if cell != "relu":  # (there the larger of NaN and 0 is 0)
        assert out[1][0][1:, 2].isnan().all() and out[1][0][:, 4].isnan().any()


@pytest.mark.parametrize("H,B", [(256, 20), (320, 5)])
def test_a_row_that_is_not_finite_spoils_no_other(H, B):
    import torch

    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.inputs import make_inputs
    from paper_1604_01946_amd.runner import LstmRunner

    c = cfg(2, 4, B, 24, H)
    d = make_inputs(c, 3)
    whole = LstmRunner(c.dims, d)
    binding.check(whole.forward())
    binding.check(whole.backward())
    d["x"][1, 2, 5] = float("nan")
    d["x"][2, 3, :] = float("inf")
    r = LstmRunner(c.dims, d)
    binding.check(r.forward())
    binding.check(r.backward())
    torch.cuda.synchronize()
    keep = [b for b in range(B) if b not in (2, 3)]
    for a, b in ((r.y, whole.y), (r.hT, whole.hT), (r.cT, whole.cT), (r.dx, whole.dx), (r.dh0, whole.dh0), (r.dc0, whole.dc0)):
        a, b = a.view(-1, B, a.shape[-1]), b.view(-1, B, b.shape[-1])
        # (not the same bits: a product that finds a sum that is not finite works its tile out with other instructions; sums
        # of up to 4 H terms, four steps)
        assert (a[:, keep] - b[:, keep]).abs().max() <= 1e-5 * b.abs().max()
    assert r.y[1:, 2].isnan().all()
    binding.check(r.forward())  # no wait expired
