"""Operands whose magnitudes lie far apart inside one row or column: every sum keeps fp32's error relative to its own terms, in the
products that callers ask for by themselves and in those inside a pass.  Reference: float64."""
import numpy as np
import pytest

from oracle import lstm_oracle as O
from paper_1604_01946_amd.inputs import Config, make_inputs
from test_gpu_gemm_split3 import check, operands, run
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu
WS = 64 << 20


# Every row has one value that is 2^30 times the others and meets zeros only, then the same for every column.
@pytest.mark.parametrize("K", [512, 6000])
@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("layout", ["NT", "TN"])
def test_large_values_that_meet_zeros(K, side, layout):
    A, Bm = operands(300, 400, K, 7)
    if side == "A":
        A[:, 77], Bm[77] = 2.0 ** 30, 0
    else:
        Bm[77], A[:, 77] = 2.0 ** 30, 0
    check(run(A, Bm, layout, scratch_bytes=WS), *((A * (np.arange(K) != 77), Bm) if side == "A" else (A, Bm * (np.arange(K) != 77)[:, None])))
    # a single row, a single column
    A, Bm = operands(300, 400, K, 7)
    A[5, 77], Bm[77] = 2.0 ** 30, 0
    A[:, 78], Bm[78, 9] = 0, -2.0 ** 31
    a, b = A.copy(), Bm.copy()
    a[5, 77] = b[78, 9] = 0
    check(run(A, Bm, layout, scratch_bytes=WS), a, b)


# The same value meets something in every 64th column, so that its row is not one of small sums only.
@pytest.mark.parametrize("M,N,K", [(512, 512, 2048), (2048, 2048, 512), (700, 652, 676)])
@pytest.mark.parametrize("layout", ["NT", "NN", "TN"])
@pytest.mark.parametrize("power", [20, 30])
def test_large_values_that_meet_a_few(M, N, K, layout, power):
    A, Bm = operands(M, N, K, 7)
    A[5, 77], Bm[77] = 2.0 ** power, 0
    Bm[77, ::64] = 1
    got = run(A, Bm, layout, scratch_bytes=WS)
    other = np.arange(N) % 64 != 0
    a = A.copy()
    a[5, 77] = 0
    check(got[:, other], a, Bm[:, other])
    check(got, A, Bm, wide=True)


# Inside a pass.  Forward: one input of 2^30 that a unit in 64 looks at; the others' pre-activations are those of the remaining
# inputs.  Backward: the upstream gradient of one row of the first step is 2^30, and an input in 64 of that row is not zero; the
# columns of dW that belong to the others are sums over the other rows.
@pytest.mark.parametrize("L,T,B,I,H", [(1, 50, 128, 1024, 1024), (1, 100, 64, 512, 512), (1, 40, 128, 512, 2048), (1, 100, 128, 1024, 512)])
def test_passes_beside_large_values(L, T, B, I, H):
    import torch
    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.runner import LstmRunner
    cfg = Config("ranges", L=L, T=T, B=B, I=I, H=H, state_std=0.3)
    print("ranges", cfg.dims, flush=True)

    def both(d):
        y, _, _, res = O.lstm_forward(*cfg.dims, d["x"], d["h0"], d["c0"], d["W"], d["R"], d["b"])
        g = O.lstm_backward(*cfg.dims, d["x"], d["h0"], d["c0"], d["W"], d["R"], res, d["dy"], None, None)
        r = LstmRunner(cfg.dims, d, with_dstates=False)
        r.poison()
        binding.check(r.forward(), "forward")
        binding.check(r.backward(), "backward")
        torch.cuda.synchronize()
        return r.y.cpu().numpy(), y, r.dW.cpu().numpy().reshape(4 * H, I), np.asarray(g[3]).reshape(4 * H, I)

    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)  # noqa: E731
    d = make_inputs(cfg, 3)
    W = d["W"].reshape(4, H, I)
    W[:, np.arange(H) % 64 != 0, 77] = 0
    d["x"][0, 5, 77] = 2.0 ** 30
    got, ref, _, _ = both(d)
    other = np.arange(H) % 64 != 0
    # (sqrt(K) 2^-24 with K of up to 2048; operands scaled to 2^30 in two fp16 parts: 1.2e-3)
    assert rel(got[0, 5, other], ref[0, 5, other]) < 5e-6
    d = make_inputs(cfg, 3)
    d["dy"][0, 5] *= 2.0 ** 30
    d["x"][0, 5, np.arange(I) % 64 != 0] = 0
    _, _, got, ref = both(d)
    other = np.arange(I) % 64 != 0
    assert rel(got[:, other], ref[:, other]) < 5e-6


@pytest.mark.parametrize("K", [900, 6000])
def test_infinities_and_nan_as_in_fp32(K):
    A, Bm = operands(300, 260, K, 4)
    Bm = np.abs(Bm) + np.float32(0.5)
    A[3, 7], A[150, K - 1], A[290, 0] = np.inf, -np.inf, np.nan
    A[7, :] = 0
    A[7, 5] = np.float32(3.4e38)
    Bm[5, :] = np.float32(0.5)
    got = run(A, Bm, "NT", scratch_bytes=WS)
    assert np.all(np.isposinf(got[3])) and np.all(np.isneginf(got[150])) and np.all(np.isnan(got[290]))
    assert np.allclose(got[7], 1.7e38, rtol=1e-6)
    rest = [i for i in range(300) if i not in (3, 150, 290, 7)]
    check(got[rest], A[rest], Bm, wide=True)


# whole passes: input products, gradients, weight gradients with and without an initial state in front of the others
@pytest.mark.parametrize("L,T,B,I,H", [(2, 3, 32, 24, 1024), (1, 3, 64, 520, 520), (2, 4, 48, 640, 640), (1, 2, 33, 64, 1280), (2, 5, 64, 256, 256)])
def test_passes(L, T, B, I, H):
    run_case(Config("ranges", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3), 3, 0)
    run_cell("gru", L, T, B, I, H, seed=4)
