"""Inference calls of one step and few rows (one launch per layer): against the oracle and against the paths for sequences, with and
without initial states, states carried in place, hidden and input sizes that allow no vector loads, both sides of the line in rows."""
import numpy as np
import pytest

from oracle import lstm_oracle as O
from paper_1604_01946_amd.inputs import Config, make_inputs
from parity import FWD_TOL, nerr

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 4, 4), (2, 1, 256, 256), (1, 2, 80, 320), (3, 3, 33, 40), (2, 4, 100, 301), (1, 5, 7, 1023), (2, 8, 650, 650), (4, 16, 64, 512),
          (2, 17, 64, 128), (1, 16, 2048, 2048), (2, 9, 3, 64)]


@pytest.mark.parametrize("L,B,I,H", SHAPES)
@pytest.mark.parametrize("states", ["none", "given", "in place"])
def test_one_step(L, B, I, H, states):
    import torch
    from paper_1604_01946_amd import binding
    cfg = Config("cell", L=L, T=1, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)
    d = make_inputs(cfg, 3)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    h0, c0 = (None, None) if states == "none" else (up(d["h0"]), up(d["c0"]))
    y, _, _ = (torch.full((1, B, H), float("nan"), device="cuda") for _ in range(3))
    hT, cT = (h0, c0) if states == "in place" else (torch.full((L, B, H), float("nan"), device="cuda") for _ in range(2))
    wb = binding.lstm_workspace_bytes(*cfg.dims)
    ws = torch.full((wb // 4,), float("nan"), device="cuda")
    x, W, R, b = (up(d[k]) for k in "xWRb")
    print("one step", cfg.dims, states, flush=True)
    ref = O.lstm_forward(*cfg.dims, d["x"], None if h0 is None else d["h0"], None if c0 is None else d["c0"], d["W"], d["R"], d["b"])
    binding.check(binding.lstm_forward(*cfg.dims, x, h0, c0, W, R, b, y, hT, cT, None, ws, wb), "lstm_forward")
    torch.cuda.synchronize()
    for got, want in ((y, ref[0]), (hT, ref[1]), (cT, ref[2])):
        assert nerr(got.cpu().numpy(), want) < FWD_TOL
    # results nobody wants; the same call again is the same bit for bit
    if states == "given":
        y2 = torch.full_like(y, float("nan"))
        binding.check(binding.lstm_forward(*cfg.dims, x, h0, c0, W, R, b, y2, None, None, None, ws, wb), "lstm_forward")
        torch.cuda.synchronize()
        assert torch.equal(y, y2)


def test_overlaps_that_it_leaves_to_the_other_paths(knobs):
    """c0 where hT goes and the other way round: as without this kernel."""
    import torch
    from paper_1604_01946_amd import binding
    cfg = Config("cell", L=2, T=1, B=4, I=64, H=128, state_std=0.3, dstate_std=0.3)
    d = make_inputs(cfg, 3)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    x, W, R, b = (up(d[k]) for k in "xWRb")
    wb = binding.lstm_workspace_bytes(*cfg.dims)
    ws = torch.empty(wb // 4, device="cuda")
    got = []
    for on in ("1", "0"):
        knobs(LSTM_CELL_STEP=on)
        h0, c0, y = up(d["h0"]), up(d["c0"]), torch.empty(1, 4, 128, device="cuda")
        cT = torch.empty_like(c0)
        binding.check(binding.lstm_forward(*cfg.dims, x, h0, c0, W, R, b, y, c0, cT, None, ws, wb), "lstm_forward")
        torch.cuda.synchronize()
        got.append((y.clone(), c0.clone(), cT.clone()))
    for p, q in zip(*got):
        assert torch.equal(p, q)


@pytest.mark.parametrize("L,B,I,H,here", [(16, 16, 128, 128, False), (8, 8, 40, 100, False), (8, 1, 256, 256, False), (4, 12, 320, 320, False),
                                          (16, 1, 128, 128, True), (8, 4, 256, 256, True), (3, 16, 64, 320, True), (12, 16, 64, 512, True)])
def test_deep_stacks_of_few_units_run_as_sequences(L, B, I, H, here):
    import torch
    from paper_1604_01946_amd import binding
    from parity import recurrence_kernels
    cfg = Config("cell", L=L, T=1, B=B, I=I, H=H, state_std=0.3)
    d = make_inputs(cfg, 3)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    x, W, R, b, h0, c0 = (up(d[k]) for k in ("x", "W", "R", "b", "h0", "c0"))
    wb = binding.lstm_workspace_bytes(*cfg.dims)
    ws, y = torch.full((wb // 4,), float("nan"), device="cuda"), torch.full((1, B, H), float("nan"), device="cuda")
    print("one step", cfg.dims, flush=True)
    kernel, _ = recurrence_kernels(lambda: binding.check(
        binding.lstm_forward(*cfg.dims, x, h0, c0, W, R, b, y, None, None, None, ws, wb), "lstm_forward"))
    assert (kernel == "lstm_cell_kernel") == here, kernel
    ref = O.lstm_forward(*cfg.dims, d["x"], d["h0"], d["c0"], d["W"], d["R"], d["b"])
    assert nerr(y.cpu().numpy(), ref[0]) < FWD_TOL
