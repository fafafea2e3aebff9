"""Kernels whose workgroups exchange a step's values through the L2 of one XCD.  A single sequence: lengths around the chunks of
steps whose reserve values pass through LDS together, one and more layers; the same bits with stores that write through to memory
(LSTM_FULL_FENCES), which is what a layer spread over XCDs uses."""
import pytest

from paper_1604_01946_amd.inputs import Config
from test_gpu_parity import BWD, FWD, run_case

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
