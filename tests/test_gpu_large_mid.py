"""One-layer kernels of hidden sizes between 512, 1024 and 2048: blocks of the backward tiles with more workgroups than finalise
(one or two octets of units each), partial sums that do not spread evenly over the counter lines (640, 768, 896, 1536, 1792), groups of K that do not divide by four (640, 896), tiles cut in four and in two, several slices and
launches, weights partly in LDS (1536, 1792); fp32 and bf16 products, repeated launches; sizes that are padded to them."""
import pytest

from paper_1604_01946_amd.inputs import Config
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu


def cfg(L, T, B, I, H):
    return Config("mid", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3)


@pytest.mark.parametrize("H", [640, 768, 896, 1536, 1792])
@pytest.mark.parametrize("split3", ["0", "1", "2"])
@pytest.mark.parametrize("L,T,B", [(1, 3, 20), (2, 4, 33), (1, 3, 64)])
def test_native(H, split3, L, T, B, knobs):
    knobs(LSTM_SPLIT3=split3)
    run_case(cfg(L, T, B, 48, H), 7, 0)


@pytest.mark.parametrize("H", [640, 768, 896])
@pytest.mark.parametrize("split3", ["0", "1"])
@pytest.mark.parametrize("L,T,B", [(1, 3, 100), (2, 3, 200), (1, 2, 256), (1, 2, 257)])
def test_several_launches(H, split3, L, T, B, knobs):
    knobs(LSTM_SPLIT3=split3)
    run_case(cfg(L, T, B, 48, H), 7, 0)


@pytest.mark.parametrize("H,B", [(513, 1), (650, 20), (700, 70), (800, 33), (897, 9), (1000, 64), (1100, 8), (1500, 30), (1537, 2), (1700, 64)])
def test_padded(H, B):
    run_case(cfg(2, 3, B, 50, H), 9, 0)


@pytest.mark.parametrize("H", [640, 768, 896, 1536, 1792, 650, 1400])
@pytest.mark.parametrize("cell", ["gru", "tanh"])
@pytest.mark.parametrize("L,T,B", [(1, 22, 3), (2, 3, 40), (3, 22, 33)])
def test_other_cells(H, cell, L, T, B):
    if L * T * H > 60000:
        T = 3
    run_cell(cell, L, T, B, 64, H, seed=4)


@pytest.mark.parametrize("H,B", [(640, 30), (768, 70), (896, 64), (1536, 32), (700, 30)])
def test_long_products(H, B):
    """1024 rows and more: weight gradients with long sums."""
    run_case(cfg(2, (1024 + B - 1) // B, B, H, H), 5, 0)
