"""GPU parity of the single-gate RNN and GRU cells: rnn_forward / rnn_backward through the C ABI against the CPU
oracle on the same seeded inputs.  Tolerances as for the LSTM: max|gpu-oracle|/max|oracle| <= 1e-4 forward, <= 1e-3
for every gradient."""
import numpy as np
import pytest

from oracle import rnn_oracle as O
from parity import assert_close, nerr, FWD_TOL, BWD_TOL

pytestmark = pytest.mark.gpu


def make(cell, L, T, B, I, H, seed, with_h0=True):
    rng = np.random.default_rng(seed)
    G = O.CELLS[cell] * H
    nw = G * I + (L - 1) * G * H
    a = 1.0 / np.sqrt(H)
    d = dict(x=rng.standard_normal((T, B, I)), W=rng.uniform(-a, a, nw), R=rng.uniform(-a, a, (L, G, H)),
             b=rng.uniform(-0.1, 0.1, (L, G)), h0=0.3 * rng.standard_normal((L, B, H)) if with_h0 else None,
             dy=rng.standard_normal((T, B, H)), dhT=0.3 * rng.standard_normal((L, B, H)) if with_h0 else None)
    return {k: (None if v is None else v.astype(np.float32)) for k, v in d.items()}


RELU_TIE = 3e-6     # ten times the fp32 rounding of these pre-activation sums
MAX_ROW_TIES = 8    # per batch row: 2^8 one-row oracle backward passes at most


def relu_ties(L, T, B, I, H, d, saved):
    """Index array [k][4] = (layer, step, batch row, unit) of the ReLU units whose pre-activation (oracle, float64)
    is within RELU_TIE of zero.  The backward pass switches on the sign of the pre-activation, and which side such
    an element is on is not decided by the fp32 arithmetic of the kernels: 0 and 1 are both correct slopes for it,
    so the network has 2^k correct gradients, and the comparison below accepts exactly those."""
    a = O.relu_preactivations(L, T, B, I, H, d["x"], d["h0"], d["W"], d["R"], d["b"], saved)
    return np.argwhere(np.abs(a) < RELU_TIE)


def relu_slopes_matching(L, T, B, I, H, d, saved, ties, got_dx, got_dh0):
    """Slope array [L][T][B][H]: the oracle's own decisions (h > 0) everywhere except at the tied units, where the
    admissible assignment (0 or 1 each) is searched for.  Batch rows do not interact in the backward recurrence, and
    dx and dh0 of a row depend on that row's slopes only, so the search runs row by row over one-row oracle
    problems: the assignment whose dx, dh0 lie nearest to the kernels' is kept.  The caller then compares EVERY
    gradient with the oracle's result for the returned assignment, so the search only chooses which of the valid
    results to compare with."""
    slope = (saved["h"] > 0).astype(np.float64)
    for b in sorted(set(int(v) for v in ties[:, 2])):
        mine = [tuple(int(v) for v in ix) for ix in ties if ix[2] == b]
        assert len(mine) <= MAX_ROW_TIES, f"batch row {b} has {len(mine)} tied units"
        row = lambda a: None if a is None else np.asarray(a, np.float64)[:, b:b + 1]
        sv = {"h": saved["h"][:, :, b:b + 1]}
        best = None
        for bits in range(1 << len(mine)):
            s1 = slope[:, :, b:b + 1].copy()
            for j, (l, t, _, u) in enumerate(mine):
                s1[l, t, 0, u] = float((bits >> j) & 1)
            dx1, dh01 = O.rnn_backward("relu", L, T, 1, I, H, row(d["x"]), row(d["h0"]), d["W"], d["R"], sv, row(d["dy"]),
                                       row(d["dhT"]), relu_slope=s1)[:2]
            err = max(nerr(got_dx[:, b:b + 1], dx1), nerr(got_dh0[:, b:b + 1], dh01))
            if best is None or err < best[0]:
                best = (err, s1)
        slope[:, :, b:b + 1] = best[1]
    return slope


def run(cell, L, T, B, I, H, seed, with_h0=True):
    import torch
    from paper_1604_01946_amd import binding as Bd
    d = make(cell, L, T, B, I, H, seed, with_h0)
    y, hT, saved = O.rnn_forward(cell, L, T, B, I, H, d["x"], d["h0"], d["W"], d["R"], d["b"])
    ties = relu_ties(L, T, B, I, H, d, saved) if cell == "relu" else np.zeros((0, 4), int)
    dev = "cuda:0"
    up = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    t = {k: up(v) for k, v in d.items()}
    c = Bd.RNN_CELLS[cell]
    f = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device=dev)
    out = dict(y=f(T, B, H), hT=f(L, B, H), dx=f(T, B, I), dh0=f(L, B, H), dW=f(d["W"].size), dR=f(*d["R"].shape), db=f(*d["b"].shape))
    rb, wb = Bd.rnn_reserve_bytes(c, L, T, B, I, H), Bd.rnn_workspace_bytes(c, L, T, B, I, H)
    res = torch.full((rb // 4,), float("nan"), dtype=torch.float32, device=dev)
    ws = torch.full((wb // 4,), float("nan"), dtype=torch.float32, device=dev)
    print(f"case {cell} {(L, T, B, I, H)} seed={seed} h0={with_h0} ties={len(ties)}", flush=True)
    Bd.check(Bd.rnn_forward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], t["b"], out["y"], out["hT"], res, ws, wb), "rnn_forward")
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    assert_close(got, dict(y=y, hT=hT), ("y", "hT"), FWD_TOL, f"fwd {cell}")
    Bd.check(Bd.rnn_backward(c, L, T, B, I, H, t["x"], t["h0"], t["W"], t["R"], res, t["dy"], t["dhT"], out["dx"], out["dh0"],
                             out["dW"], out["dR"], out["db"], ws, wb), "rnn_backward")
    torch.cuda.synchronize()
    names = ("dx", "dh0", "dW", "dR", "db")
    got = {k: out[k].cpu().numpy() for k in names}
    slope = None
    if cell == "relu" and len(ties):  # which of the 2^k valid gradients the kernels produced
        slope = relu_slopes_matching(L, T, B, I, H, d, saved, ties, got["dx"].reshape(T, B, I), got["dh0"].reshape(L, B, H))
    kw = {} if slope is None else {"relu_slope": slope}
    ref = dict(zip(names, O.rnn_backward(cell, L, T, B, I, H, d["x"], d["h0"], d["W"], d["R"], saved, d["dy"], d["dhT"], **kw)))
    got = {k: got[k].reshape(np.asarray(ref[k]).shape) for k in names}
    assert_close(got, ref, names, BWD_TOL, f"bwd {cell} ({len(ties)} tied slopes)")


SHAPES = [(1, 8, 4, 32, 32), (3, 5, 7, 24, 40), (2, 6, 64, 128, 256), (4, 12, 33, 512, 512), (1, 1, 1, 16, 16), (2, 3, 3, 5, 7)]


@pytest.mark.parametrize("cell", ["relu", "tanh", "gru"])
@pytest.mark.parametrize("dims", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_cells_match_oracle(cell, dims):
    run(cell, *dims, seed=3)


# Hidden sizes below 512 without persistent kernels run zero-padded to 128 / 256 / 512 (as the LSTM's do);
# RNN_NO_PERSISTENT=1 runs them as given on the step-by-step path, which keeps its ragged tiles covered.
# (between 1024 and 2048 with few rows: padded to 2048)
RAGGED = [(3, 5, 7, 24, 40), (2, 3, 3, 5, 7), (2, 4, 70, 36, 100), (2, 40, 9, 300, 300), (2, 3, 9, 64, 600), (2, 2, 12, 48, 1500)]


@pytest.mark.parametrize("step_by_step", [False, True], ids=["padded", "as_given"])
@pytest.mark.parametrize("cell", ["relu", "tanh", "gru"])
@pytest.mark.parametrize("dims", RAGGED, ids=["x".join(map(str, s)) for s in RAGGED])
def test_ragged_hidden_sizes(cell, dims, step_by_step, knobs):
    if step_by_step:
        knobs(RNN_NO_PERSISTENT="1")
    run(cell, *dims, seed=11)


@pytest.mark.parametrize("cell", ["tanh", "gru"])
def test_measured_shape_at_full_size(cell):
    """The shape the cells are timed at (four layers, H = 512, minibatch 64, 100 steps: the paper's LSTM shape),
    compared element by element."""
    run(cell, 4, 100, 64, 512, 512, seed=1)


@pytest.mark.parametrize("cell", ["tanh", "gru"])
def test_cells_without_initial_state(cell):
    run(cell, 2, 4, 5, 16, 48, seed=4, with_h0=False)


# Shapes the persistent kernels take (H in 128/256/512), all three cells: x multiplied inside the kernel
# (I == H) or projected by a batched GEMM (I != H), batch slices side by side and in further launches, a single step.
PERSISTENT = [(4, 7, 64, 512, 512), (2, 5, 33, 72, 256), (3, 4, 130, 128, 128), (1, 3, 48, 512, 512), (2, 1, 64, 256, 256),
              (1, 2, 512, 16, 128), (2, 6, 32, 256, 256), (4, 5, 1, 512, 512), (3, 4, 17, 40, 128),
              (3, 3, 130, 256, 256),   # three slices of 64 rows, two side by side and one in a second launch
              (1, 2, 600, 16, 128)]    # ten slices (GRU; the single gate runs this batch step by step)


@pytest.mark.parametrize("with_h0", [True, False], ids=["h0", "noh0"])
@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("dims", PERSISTENT, ids=["x".join(map(str, s)) for s in PERSISTENT])
def test_persistent_shapes(dims, cell, with_h0):
    run(cell, *dims, seed=5, with_h0=with_h0)


# Beyond one launch of 16-row slices the GRU runs on the kernels with two alternating chains per slice (where x is multiplied inside the
# kernel, I == H, forward; always backward), and with LSTM_NEAR=0 every cell does (test_gpu_step_counters.py); RNN_PINGPONG=0 keeps the one-chain kernels covered at those shapes.
@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("dims", [PERSISTENT[0], PERSISTENT[1], PERSISTENT[3], PERSISTENT[7], PERSISTENT[9]],
                         ids=["4x7x64x512x512", "2x5x33x72x256", "1x3x48x512x512", "4x5x1x512x512", "3x3x130x256x256"])
def test_cells_on_the_one_chain_kernels(dims, cell, knobs):
    knobs(RNN_PINGPONG="0")
    run(cell, *dims, seed=6)


# Stacks deeper than the chip holds at once: groups of consecutive layers, one launch per group
DEEP = [(5, 4, 64, 512, 512), (6, 3, 130, 512, 512), (9, 3, 20, 48, 256), (17, 2, 8, 128, 128)]


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("dims", DEEP, ids=["x".join(map(str, s)) for s in DEEP])
def test_persistent_layer_groups(dims, cell):
    run(cell, *dims, seed=9)


# Large hidden sizes: the one-layer persistent kernels (recurrent matrix spread over all CUs), slices of 32 batch rows
LARGE = [(2, 4, 32, 96, 1024), (1, 3, 64, 1024, 1024), (1, 3, 100, 64, 1024), (1, 2, 8, 128, 2048), (1, 2, 16, 64, 1024),
         (2, 1, 5, 2048, 2048), (1, 2, 40, 64, 2048)]


@pytest.mark.parametrize("with_h0", [True, False], ids=["h0", "noh0"])
@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
@pytest.mark.parametrize("dims", LARGE, ids=["x".join(map(str, s)) for s in LARGE])
def test_large_hidden_shapes(dims, cell, with_h0):
    run(cell, *dims, seed=8, with_h0=with_h0)


@pytest.mark.parametrize("cell", ["gru", "tanh", "relu"])
def test_step_by_step_path_at_a_persistent_shape(cell, knobs):
    knobs(RNN_NO_PERSISTENT="1")
    run(cell, 2, 5, 40, 64, 128, seed=6)
