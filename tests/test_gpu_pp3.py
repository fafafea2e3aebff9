"""The alternating persistent kernels on the bf16 matrix cores (operands in three parts): every hidden size and cell they
take, batches that end inside a chain, inputs narrower than the hidden size, one step, several slices and launches; and what
an infinite, NaN or very large operand gives, which has to be what the fp32 kernels give (LSTM_PINGPONG=0 / RNN_PINGPONG=0)."""
import numpy as np
import pytest

from paper_1604_01946_amd.inputs import Config, make_inputs
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu

LSTM = [Config(f"pp3-{L}-{T}-{B}-{I}-{H}", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)
        for L, T, B, I, H in [(2, 1, 33, 128, 128), (2, 1, 33, 256, 256), (2, 2, 64, 100, 256), (3, 5, 65, 256, 256), (1, 3, 129, 17, 256),
                              (4, 6, 50, 512, 512), (2, 4, 64, 511, 512), (1, 3, 200, 512, 512), (5, 3, 40, 512, 512)]]


@pytest.mark.parametrize("cfg", LSTM, ids=lambda c: c.name)
def test_lstm(cfg):
    run_case(cfg, 3, 0)


@pytest.mark.parametrize("cell", ["gru", "tanh"])
@pytest.mark.parametrize("shape", [(2, 1, 20, 256, 256), (2, 4, 33, 256, 256), (3, 3, 64, 100, 256), (4, 5, 70, 512, 512)])
def test_cells(cell, shape):
    run_cell(cell, *shape, seed=5)


@pytest.mark.parametrize("where", ["x", "h0", "W", "R", "dy"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_operands_without_parts(where, value, knobs):
    import torch
    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.runner import LstmRunner
    cfg = Config("odd", L=2, T=4, B=48, I=256, H=256, state_std=0.3, dstate_std=0.3)
    d = make_inputs(cfg, 1)
    d[where].reshape(-1)[d[where].size // 2 + 3] = value
    got = []
    for setting in (None, "0"):
        knobs(LSTM_PINGPONG=setting)
        r = LstmRunner(cfg.dims, d)
        for _ in range(2):  # the second call finds nothing of the first
            r.poison()
            binding.check(r.forward(), "forward")
            binding.check(r.backward(), "backward")
        torch.cuda.synchronize()
        got.append({**r.fwd_outputs(), **r.bwd_outputs()})
    for k in got[0]:
        a, b = got[0][k].astype(np.float64), got[1][k].astype(np.float64)
        fine = np.isfinite(b)
        # (an infinite sum may come out NaN or infinite by the order of its terms: finite or not is what is compared)
        assert np.array_equal(np.isfinite(a), fine), (k, np.isfinite(a).sum(), fine.sum())
        if fine.any():
            scale = np.max(np.abs(b[fine]))
            assert np.max(np.abs(a[fine] - b[fine])) <= 1e-4 * scale, k
