"""The GEMM on fp16 matrix cores (operands in two parts, scaled row by row) at the sizes where it can go wrong: edges of the 128 and
256 tiles, K around multiples of its k-tile of 32, K slices, rows and columns of zeros, magnitudes far apart, operands near the
bottom and the top of the fp32 range, infinities and NaN.  Reference: float64.

LSTM_GEMM_HALF=1 sends every product here that has 16-byte aligned rows and scratch for the largest magnitudes."""
import numpy as np
import pytest

from paper_1604_01946_amd.inputs import Config
from test_gpu_gemm_split3 import check, operands, run
from test_gpu_parity import run_case
from test_gpu_rnn_cells import run as run_cell

pytestmark = pytest.mark.gpu
WS = 64 << 20


@pytest.fixture(autouse=True)
def all_here(knobs):
    knobs(LSTM_GEMM_SHORT="0", LSTM_GEMM_HALF="1")


@pytest.mark.parametrize("M,N,K", [(4, 4, 4), (12, 20, 28), (124, 132, 32), (128, 128, 36), (260, 256, 60), (252, 516, 64), (700, 652, 676),
                                   (1100, 2052, 40), (3600, 4100, 92), (3596, 4096, 128)])
@pytest.mark.parametrize("layout", ["NT", "NN", "TN", "TT"])
def test_edges(M, N, K, layout):
    A, Bm = operands(M, N, K, M + N + K)
    check(run(A, Bm, layout, scratch_bytes=WS), A, Bm)
    if M * N < 10 ** 6:
        C0 = np.random.default_rng(6).standard_normal((M, N)).astype(np.float32)
        check(run(A, Bm, layout, accumulate=1, scratch_bytes=WS, C0=C0), A, Bm, C0)


# (rows that do not divide by four where they are not the unit stride; no scratch: three bf16 parts)
@pytest.mark.parametrize("M,N,K", [(9, 7, 100), (255, 514, 1000), (1030, 641, 1996)])
@pytest.mark.parametrize("scratch", [0, 4096, WS])
def test_ragged_rows(M, N, K, scratch):
    A, Bm = operands(M, N, K, 3)
    check(run(A, Bm, "NT", scratch_bytes=scratch), A, Bm)


@pytest.mark.parametrize("M,N,K", [(512, 512, 4000), (132, 260, 8200), (2048, 1028, 2400)])
@pytest.mark.parametrize("layout", ["NT", "NN", "TN"])
def test_slices(M, N, K, layout):
    A, Bm = operands(M, N, K, 5)
    C0 = np.random.default_rng(6).standard_normal((M, N)).astype(np.float32)
    got = run(A, Bm, layout, accumulate=1, scratch_bytes=WS, C0=C0)
    check(got, A, Bm, C0)
    assert np.array_equal(got, run(A, Bm, layout, accumulate=1, scratch_bytes=WS, C0=C0))


# One term per sum: an operand is off by up to 2^-23 of itself, the product of the remainders that is left out is up to 2^-22 of
# the whole, and two of the three additions cost 2^-23 of it each: 2^-20.4 at the very worst (three bf16 parts: 2^-22.4; rms 2^-23.5 and
# 2^-24.8).  Values below 2^-18 of the largest of their row or column end at 2^-40 of it, times 2^-24 / 2^-25 there.
@pytest.mark.parametrize("M,N,K", [(700, 652, 652), (512, 512, 4000), (2048, 1028, 2400), (3600, 4100, 140)])
@pytest.mark.parametrize("layout", ["NT", "NN", "TN"])
def test_one_term(M, N, K, layout):
    A, Bm = operands(M, N, K, 8)
    at = np.random.default_rng(9).integers(0, K, M)
    term = A[np.arange(M), at][:, None].astype(np.float64) * Bm[at].astype(np.float64)
    A *= np.arange(K)[None] == at[:, None]
    got = run(A, Bm, layout, scratch_bytes=WS)
    floor = np.abs(A[np.arange(M), at])[:, None] * np.abs(Bm).max(0)[None] * 2.0 ** -39
    assert np.all(np.abs(got - term) <= np.abs(term) * 2.0 ** -20.4 + floor)


# The same tile and slices of the same length, three additions per 16 k where six were made: measured 0.73 times the error.
@pytest.mark.parametrize("M,N,K,layout", [(4096, 4096, 1024, "NT"), (4096, 4096, 1024, "NN"), (4096, 4096, 2048, "TN"), (2048, 4096, 512, "NN")])
def test_errors_are_smaller_than_with_three_bf16_parts(M, N, K, layout, knobs):
    A, Bm = operands(M, N, K, 12)
    ref = A.astype(np.float64) @ Bm.astype(np.float64)
    e = []
    for half in ("1", "0"):
        knobs(LSTM_GEMM_HALF=half, LSTM_GEMM_SPLIT="0")
        e.append(np.linalg.norm(run(A, Bm, layout, scratch_bytes=WS) - ref))
    assert e[0] < 0.85 * e[1]


# Every row has one value that is 2^30 times the others and meets zeros only, then the same for every column: scaled to the large
# value the others have few bits left, and the sums are worked out again.
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


def test_zeros():
    A, Bm = operands(300, 520, 300, 2)
    A[7] = A[256:] = 0
    Bm[:, 3] = Bm[:, 256:512] = 0
    check(run(A, Bm, "NT", scratch_bytes=WS), A, Bm)
    assert not run(A * 0, Bm, "TN", scratch_bytes=WS).any()


@pytest.mark.parametrize("exponent", [-112, -125, -132])
@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("M,N,K", [(260, 132, 516), (128, 256, 4096), (4096, 4096, 272)])
def test_small_operands(M, N, K, exponent, side):
    A, Bm = operands(M, N, K, 4)
    tiny, other = np.float64(2.0) ** exponent, 2.0 ** 30
    A, Bm = (A * (tiny if side == "A" else other)).astype(np.float32), (Bm * (tiny if side == "B" else other)).astype(np.float32)
    got, ref = run(A, Bm, "NT", scratch_bytes=WS), A.astype(np.float64) @ Bm.astype(np.float64)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 2.0 ** -24 * np.sqrt(K) + 2.0 ** -23


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


def test_sums_of_results_are_not_biased():
    for layout in ("NT", "NN", "TN"):
        A, Bm = operands(4096, 3072, 1024, 17)
        ref = A.astype(np.float64) @ Bm.astype(np.float64)
        e = (run(A, Bm, layout, scratch_bytes=WS) - ref) / np.sqrt(np.mean(ref ** 2))
        for block in (e, e[:, :256], e[:, 512:513], e[:256], e[7:8]):
            assert abs(block.mean()) < 1e-8 + 5 * 5e-7 / np.sqrt(block.size)


# whole passes: input products, gradients, weight gradients with and without a head (an initial state) of whole k-tiles
@pytest.mark.parametrize("L,T,B,I,H", [(2, 3, 32, 24, 1024), (1, 3, 64, 520, 520), (2, 4, 48, 640, 640), (1, 2, 33, 64, 1280), (2, 5, 64, 256, 256)])
def test_passes(L, T, B, I, H):
    run_case(Config("split2", L=L, T=T, B=B, I=I, H=H, state_std=0.3, dstate_std=0.3), 3, 0)
    run_cell("gru", L, T, B, I, H, seed=4)
