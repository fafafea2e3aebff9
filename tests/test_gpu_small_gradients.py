"""Weight gradients of upstream gradients far below one (a loss averaged over all steps and rows), every layer by itself and
relative to its own size: deep stacks that run as groups of layers on different kernels, and both kinds of stack that do
not.  The backward pass is linear in the upstream gradients, so one float64 result serves every power of two."""
import numpy as np
import pytest

from paper_1604_01946_amd.inputs import Config
from parity import oracle_results

pytestmark = pytest.mark.gpu

# Sums of T B <= 1280 terms: 2^-24 of a partial sum each, of either sign, is 2.1e-6 of the whole; the recurrence adds a few more such
# steps to the terms themselves.  Measured: up to 9e-7.
TOL = 1e-5


@pytest.mark.parametrize("L,T,B,H", [(5, 16, 64, 512), (6, 16, 80, 384), (5, 32, 33, 448), (4, 16, 64, 512), (2, 33, 32, 1024)])
def test_weight_gradients(L, T, B, H):
    import torch
    from paper_1604_01946_amd import binding
    from paper_1604_01946_amd.runner import LstmRunner
    cfg = Config("small gradients", L=L, T=T, B=B, I=H, H=H, state_std=0.3)
    d, ref = oracle_results(cfg, 6, with_dstates=False)
    r = LstmRunner(cfg.dims, d, with_dstates=False)
    r.poison()
    print("small gradients", cfg.dims, flush=True)
    binding.check(r.forward(), "forward")
    for scale in (2.0 ** -17, 2.0 ** -27):
        r.dy.copy_(torch.from_numpy(d["dy"] * np.float32(scale)))
        binding.check(r.backward(), "backward")
        torch.cuda.synchronize()
        got = r.bwd_outputs()
        for k in ("dW", "dR", "db"):
            for l in range(L):
                a, b = (np.asarray(v, np.float64).reshape(L, -1)[l] for v in (got[k], ref[k]))
                assert np.linalg.norm(a / scale - b) < TOL * np.linalg.norm(b), (k, l, scale)
