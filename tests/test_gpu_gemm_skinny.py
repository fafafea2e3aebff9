"""Products of up to 64 rows on the kernel whose operands go from memory to registers: remainders of its tiles of rows and blocks of 64
columns, K from one unit of 32 to several slices, both layouts of B, strided operands and results, values that are not finite.  What
runs on it by itself depends on models of times: LSTM_GEMM_SKINNY=2 and above runs whatever it can take, in a given number of slices."""
import pytest

pytestmark = pytest.mark.gpu

M_ = (1, 5, 15, 17, 32, 33, 49, 64)


def product(M, N, K, kn, acc=0, scratch=True, pad=8, poison=None):
    import torch

    from paper_1604_01946_amd import binding

    g = torch.Generator().manual_seed(M * 1000 + N + K)
    A = torch.randn(M, K + pad, generator=g).cuda()
    B = torch.randn((K, N + pad) if kn else (N, K + pad), generator=g).cuda()
    C = torch.randn(M, N + 3, generator=g).cuda()
    if poison is not None:
        A[0, min(3, K - 1)] = poison
    a, b = A[:, :K].double(), (B[:, :N].double() if kn else B[:, :K].double().t())
    ref = a @ b + (C[:, :N].double() if acc else 0)
    bound = a.abs() @ b.abs() + C[:, :N].abs().double()
    edge = C[:, N:].clone()
    part = torch.empty(64 << 20, dtype=torch.uint8, device="cuda") if scratch else None
    sb = (N + pad, 1) if kn else (1, K + pad)
    binding.check(binding.lstm_gemm_f32_ws(M, N, K, A, K + pad, 1, B, *sb, C, N + 3, acc, part, part.numel() if scratch else 0))
    torch.cuda.synchronize()
    assert torch.equal(C[:, N:], edge)
    return C[:, :N].double(), ref, bound


# An error of half a unit in the last place per product and per addition of partial sums, random signs: below 2^-24 sqrt(K) of the sum of
# magnitudes divided by sqrt(K); 2^-21 of the sum of magnitudes is eight times the largest single error.
@pytest.mark.parametrize("kn", [False, True])
@pytest.mark.parametrize("M", M_)
@pytest.mark.parametrize("N,K", [(64, 32), (100, 96), (1028, 512), (640, 2592), (4096, 1024), (68, 8192)])
def test_against_float64(M, N, K, kn):
    for acc in (0, 1):
        c, ref, bound = product(M, N, K, kn, acc)
        assert ((c - ref).abs() <= 2.0 ** -21 * bound).all()


# On that kernel for certain (other bits than without it): all numbers of row tiles, whole and not; a last block of 64 columns that is full,
# nearly empty and over half full; waves without any k, slices without any; without and with scratch for the slices.
@pytest.mark.parametrize("kn", [False, True])
@pytest.mark.parametrize("M", [1, 8, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("N,K,knob", [(64, 32, 2), (68, 96, 3), (100, 224, 4), (128, 256, 2), (64, 288, 5), (68, 96, 18), (132, 2048, 10), (324, 992, 18)])
def test_every_product_that_it_takes(M, N, K, knob, kn, knobs):
    import torch

    N = N if kn or N % 64 == 0 else N - 3
    knobs(LSTM_GEMM_SKINNY=knob)
    for acc in (0, 1):
        c, ref, bound = product(M, N, K, kn, acc)
        assert ((c - ref).abs() <= 2.0 ** -21 * bound).all()
    whole, ref, bound = product(M, N, K, kn, scratch=False)
    assert ((whole - ref).abs() <= 2.0 ** -21 * bound).all()
    knobs(LSTM_GEMM_SKINNY="0")
    assert not torch.equal(c, product(M, N, K, kn, 1)[0])


def error(M, N, K, kn):
    c, ref, _ = product(M, N, K, kn)
    return ((c - ref).norm() / ref.norm()).item()


# Products that fp32 instructions form (up to 8 rows with both operands contiguous along K, short ones) and products of tiles in
# three parts: with this kernel in the place of some of them no error is larger.  The norms of 10000 elements and more scatter by
# less than 1 % each; 3 % is three times the scatter of their ratio.
@pytest.mark.parametrize("M,N,K,kn", [(5, 16384, 4096, False), (8, 16384, 4096, False), (5, 2560, 640, False), (8, 2560, 640, False), (8, 8192, 2048, False),
                                      (16, 2048, 256, True), (33, 1024, 256, False), (12, 4096, 384, False), (16, 2048, 2048, False), (64, 4096, 4096, True),
                                      (16, 1024, 960, True), (8, 1024, 960, True), (32, 640, 704, True), (16, 1024, 1152, False)])
def test_no_larger_error_than_without(M, N, K, kn, knobs):
    got = error(M, N, K, kn)
    knobs(LSTM_GEMM_SKINNY="0")
    assert got <= 1.03 * error(M, N, K, kn)


@pytest.mark.parametrize("kn", [False, True])
def test_without_scratch(kn):
    c, ref, bound = product(40, 512, 4096, kn, scratch=False)
    assert ((c - ref).abs() <= 2.0 ** -21 * bound).all()


@pytest.mark.parametrize("kn", [False, True])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38])
def test_values_that_are_not_finite(kn, value, knobs):
    import torch

    knobs(LSTM_GEMM_SKINNY="2")
    c, ref, bound = product(20, 256, 1024, kn, poison=value)
    if value == 3e38:  # finite, above what the parts hold
        ok = ref.abs() <= 3.4e38
        assert ((c - ref).abs() <= 2.0 ** -21 * bound)[ok].all() and c[~ok].isinf().all()
    else:
        assert torch.equal(c[0].isnan(), ref[0].isnan()) and torch.equal(c[0].isinf(), ref[0].isinf())
        assert (c[0][ref[0].isinf()] == ref[0][ref[0].isinf()]).all()
    assert ((c - ref).abs() <= 2.0 ** -21 * bound)[1:].all()
