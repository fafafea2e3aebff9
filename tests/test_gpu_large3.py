"""The one-layer persistent kernels of H = 1024 / 2048 on the bf16 matrix cores (operands in three parts): batches on both
sides of the row count from which the backward kernel's third part has room, every split of its tiles' K, several slices and
launches, a padded hidden size, one step; and what an infinite, NaN or very large operand gives, which has to be what the
step-by-step path gives (a launch with such a sum is repeated by the fp32 kernel)."""
import numpy as np
import pytest

from paper_1604_01946_amd.inputs import Config, make_inputs
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu

SHAPES = [Config(f"large3-{L}-{T}-{B}-{I}-{H}", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)
          for L, T, B, I, H in [(1, 1, 11, 24, 1024), (1, 3, 10, 24, 1024), (1, 9, 11, 24, 1024), (2, 6, 31, 1024, 1024), (1, 5, 64, 40, 1024),
                                (3, 4, 65, 1024, 1024), (2, 3, 130, 64, 1024), (2, 7, 20, 650, 650), (1, 3, 10, 64, 2048), (2, 5, 33, 64, 2048)]]


@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: c.name)
def test_lstm(cfg):
    run_case(cfg, 3, 0)


@pytest.mark.parametrize("cell", ["gru", "relu", "tanh"])
@pytest.mark.parametrize("shape", [(2, 5, 20, 96, 1024), (1, 3, 50, 96, 1024), (2, 3, 100, 1024, 1024), (1, 4, 24, 96, 2048)])
def test_cells(cell, shape):
    run_cell(cell, *shape, seed=5)


@pytest.mark.parametrize("B,H", [(24, 1024), (40, 1024), (72, 1024), (24, 2048)])
@pytest.mark.parametrize("where", ["h0", "R", "dy"])
@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
def test_operands_without_parts(B, H, where, value):
    import torch
    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.runner import LstmRunner
    cfg = Config("odd", L=1, T=3, B=B, I=32, H=H, state_std=0.3, dstate_std=0.3)
    d = make_inputs(cfg, 1)
    d[where].reshape(-1)[d[where].size // 2 + 3] = value
    got = []
    for path in (binding.LSTM_PATH_PERSISTENT, binding.LSTM_PATH_STEP):
        r = LstmRunner(cfg.dims, d)
        for _ in range(2):  # the second call finds nothing of the first
            r.poison()
            binding.check(r.forward(flags=path), "forward")
            binding.check(r.backward(flags=path), "backward")
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
