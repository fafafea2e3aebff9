"""Hidden sizes between 128, 256 and 512: kernels for every multiple of 64, whose K quarters and counter lines are no powers of
two.  At the size itself, one below it (padded by a column) and one above the size before it; few rows (slices of 16 rows; the narrow kernels in test_gpu_step_counters.py),
slices of 16 and 64 rows, several launches, inputs wider than the hidden size, short and long enough for every variant."""
import pytest

from paper_1604_01946_amd.inputs import Config
from parity import BWD_TOL, FWD_TOL, assert_close, oracle_results, recurrence_kernels
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu

SIZES = (192, 320, 384, 448)


def cfg(L, T, B, I, H):
    return Config("granular", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)


@pytest.mark.parametrize("H", SIZES)
@pytest.mark.parametrize("split3", ["0", "1"])
@pytest.mark.parametrize("L,T,B,I", [(2, 6, 70, 48), (1, 4, 300, 0), (3, 5, 64, 0), (2, 9, 33, 600)])
def test_wide(H, split3, L, T, B, I, knobs):
    knobs(LSTM_SPLIT3=split3)
    run_case(cfg(L, T, B, I or H, H), 7, 0)


@pytest.mark.parametrize("H", SIZES)
@pytest.mark.parametrize("L,T,B,I", [(2, 5, 2, 40), (1, 20, 16, 0), (3, 5, 17, 0), (1, 9, 64, 30), (2, 4, 32, 700)])
def test_narrow(H, L, T, B, I):
    run_case(cfg(L, T, B, I or H, H), 8, 0)


@pytest.mark.parametrize("H", [129, 191, 193, 257, 319, 321, 383, 385, 447, 449, 511])
@pytest.mark.parametrize("B", [1, 20, 65])
def test_padded(H, B):
    run_case(cfg(2, 4, B, 50, H), 9, 0)


@pytest.mark.parametrize("H", SIZES + (300,))
@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("L,T,B,I", [(1, 3, 1, 20), (2, 12, 70, 0), (1, 10, 40, 500), (8, 3, 20, 0)])
def test_other_cells(H, cell, L, T, B, I):
    run_cell(cell, L, T, B, I or H, H, seed=4)


@pytest.mark.parametrize("H", SIZES)
def test_one_chain(H, knobs):
    knobs(LSTM_PINGPONG="0", RNN_PINGPONG="0")
    run_case(cfg(2, 5, 70, 48, H), 5, 0)
    run_cell("gru", 2, 5, 70, 48, H, seed=4)


def test_scratch_line_of_many_workgroups():
    """The stores that nobody wants go to a line per workgroup behind the scratch area: 256 workgroups and a batch of one."""
    run_cell("gru", 16, 3, 1, 128, 128, seed=4)


# More than 512 rows at 320 and 384, which are not padded: short passes run off the chip, longer ones on it.
@pytest.mark.parametrize("H", (320, 384))
@pytest.mark.parametrize("L,T,B,path", [(4, 1, 1024, "off"), (2, 2, 600, "off"), (2, 24, 600, "on"), (1, 16, 1030, "on")])
def test_many_rows(H, L, T, B, path):
    from paper_1604_01946_amd import binding
    for backward in (0, 1):
        assert (binding.lstm_auto_path(L, T, B, 64, H, backward) == binding.LSTM_PATH_PERSISTENT) == (path == "on")
    run_case(cfg(L, T, B, 64, H), 3, 0)
    run_cell("gru", L, T, B, 64, H, seed=4)


# One direction on chip, the other not: a reserve of either is read by the other.
@pytest.mark.parametrize("L,T,B,H,on", [(2, 8, 513, 384, (False, True)), (3, 14, 513, 384, (True, False))])
def test_many_rows_in_one_direction(L, T, B, H, on):
    from paper_1604_01946_amd import binding
    assert tuple(binding.lstm_auto_path(L, T, B, 64, H, k) == binding.LSTM_PATH_PERSISTENT for k in (0, 1)) == on
    run_case(cfg(L, T, B, 64, H), 3, 0)


# A few steps of one LSTM layer at a size with kernels of its own: both sides of the lines between them and the steps one by one.
@pytest.mark.parametrize("T,B,H,path", [(1, 20, 192, "off"), (2, 20, 192, "on"), (2, 1, 192, "off"), (3, 256, 192, "on"), (3, 257, 192, "off"),
                                        (4, 1, 320, "on"), (2, 129, 320, "on"), (4, 385, 384, "on"), (4, 300, 448, "on"), (7, 385, 448, "off")])
def test_short_passes(T, B, H, path):
    from paper_1604_01946_amd import binding
    for backward in (0, 1):
        assert (binding.lstm_auto_path(1, T, B, 64, H, backward) == binding.LSTM_PATH_PERSISTENT) == (path == "on")
    run_case(cfg(1, T, B, 64, H), 3, 0)
    for cell in ("gru", "tanh"):
        run_cell(cell, 1, T, B, 64, H, seed=4)


# One workgroup per pass or the kernels that overlap the layers: both sides of the line.
@pytest.mark.parametrize("L,T,B,H", [(4, 40, 1, 32), (4, 90, 1, 32), (2, 30, 7, 16), (2, 60, 7, 16)])
def test_micro_line(L, T, B, H):
    run_case(cfg(L, T, B, H, H), 3, 0)


# Tiny networks beyond that line: the step path still is one workgroup and the other rungs run as given, whatever the automatic choice does;
# a reserve of any path is read by the backward pass of any other.
@pytest.mark.parametrize("L,T,B,I,H", [(4, 40, 1, 24, 32), (2, 60, 7, 16, 16)])
def test_tiny_networks_on_named_paths(L, T, B, I, H, knobs):
    import torch
    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.runner import LstmRunner

    c, micro = cfg(L, T, B, I, H), ("lstm_micro_fwd_kernel", "lstm_micro_bwd_kernel")
    d, ref = oracle_results(c, 3)
    assert binding.lstm_auto_path(*c.dims, 0) == binding.LSTM_PATH_PERSISTENT

    def both(f, b):
        r = LstmRunner(c.dims, d)
        r.poison()
        print(c.dims, f, b, flush=True)
        names = recurrence_kernels(lambda: (binding.check(r.forward(flags=f)), binding.check(r.backward(flags=b))))
        assert_close(r.fwd_outputs(), ref, ("y", "hT", "cT"), FWD_TOL, f"{f}")
        assert_close(r.bwd_outputs(), ref, ("dx", "dh0", "dc0", "dW", "dR", "db"), BWD_TOL, f"{b}")
        return names

    for f in range(7):
        for b in range(7):
            names = both(f, b)
            assert (f != binding.LSTM_PATH_STEP or names[0] == micro[0]) and (b != binding.LSTM_PATH_STEP or names[1] == micro[1])
    for k in (0, 1):
        binding.check(binding.lstm_set_path(*c.dims, k, binding.LSTM_PATH_STEP))
    assert both(0, 0) == micro
    knobs(LSTM_NO_PAD="1")  # (and without kernels for the padded size)
    assert both(0, 0) == micro
