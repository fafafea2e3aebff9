"""Work that a user of this library has it do, as cases that can be measured.

Every case is one call of lstm_forward / rnn_forward (an inference pass: no reserve is kept) or a training pass
(forward with a reserve, then lstm_backward / rnn_backward), through the ctypes binding, on device tensors that the
caller keeps.  Sizes are those of the shipped configurations (`paper_1604_01946_amd/inputs.py`), of the sweeps over
hidden size and minibatch (`paper_1604_01946_amd/sweep.py`) and of the tests' ragged shapes.  All tensors are fp32: the
library has no other data type.  Of the single-gate cells only tanh is listed: with ReLU an element whose
pre-activation is within rounding of zero has two correct gradients, so two correct runs may differ.
"""
import math

import torch

from paper_1604_01946_amd import binding as lib

GATES = {"lstm": 4, "gru": 3, "tanh": 1}


def _case(name, cell, train, L, T, B, I, H):
    c = {"cell": cell, "train": train, "L": L, "T": T, "B": B, "I": I, "H": H}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one frame of one stream with the states carried by the caller (online decoding): nothing but latency
        _case("lstm-stream-step", "lstm", False, 2, 1, 1, 256, 256),
        # the smallest training call: a few short sequences through a tiny network
        _case("lstm-tiny-train", "lstm", True, 1, 8, 4, 32, 32),
        # one long sequence, a batch of one: a chain of 500 dependent steps
        _case("lstm-long-b1-train", "lstm", True, 2, 500, 1, 256, 256),
        # scoring a ragged batch: no size is a power of two or a multiple of 16
        _case("lstm-ragged-infer", "lstm", False, 3, 40, 17, 120, 300),
        # the library's headline shape: four layers of 512, minibatch 64, 100 steps
        _case("lstm-512-train", "lstm", True, 4, 100, 64, 512, 512),
        # a word-level language model of the usual odd width with a small minibatch and truncated back-propagation
        _case("lstm-650-train", "lstm", True, 2, 35, 20, 650, 650),
        # acoustic features (80 inputs) in a large odd minibatch: wide batch, narrow input
        _case("lstm-b500-train", "lstm", True, 2, 50, 500, 80, 320),
        # one layer of 1024 with two slices of 64 sequences
        _case("lstm-1024-train", "lstm", True, 1, 100, 128, 1024, 1024),
        # four layers of 2048: a recurrent matrix that fills the chip
        _case("lstm-2048-train", "lstm", True, 4, 50, 32, 2048, 2048),
        # the largest: a recurrent matrix that does not fit on chip
        _case("lstm-4096-train", "lstm", True, 1, 100, 64, 4096, 4096),
        # the other cells that the library has
        _case("gru-512-train", "gru", True, 4, 100, 64, 512, 512),
        _case("tanh-256-train", "tanh", True, 4, 100, 128, 256, 256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the same ranges: hidden sizes 16 to 4096 (half of them the powers of two that most networks
    use), 1 to 512 sequences of 1 to 500 steps, one to four layers, every cell, both directions."""
    top = work(_case("", "lstm", True, 1, 100, 64, 4096, 4096))["flops"]
    while True:
        cell = rng.choice(("lstm", "lstm", "lstm", "lstm", "gru", "tanh"))
        train = rng.random() < 0.65
        H = 2 ** rng.randint(4, 12) if rng.random() < 0.5 else _log_int(rng, 16, 4096)
        I = H if rng.random() < 0.5 else _log_int(rng, 16, 1024)
        c = _case("", cell, train, rng.randint(1, 4), _log_int(rng, 1, 500), _log_int(rng, 1, 512), I, H)
        # no dearer than the largest listed case: in arithmetic (short of its efficiency), in dependent steps, in memory
        if work(c)["flops"] > top / 4 or c["L"] * c["T"] > (500 if H > 512 or cell != "lstm" else 1000):
            continue
        if c["L"] * c["T"] * c["B"] * H > 100 * 64 * 4096 * 2:
            continue
        return c


def _sizes(case):
    L, T, B, I, H = (case[k] for k in "LTBIH")
    G = GATES[case["cell"]] * H
    return L, T, B, I, H, G, G * I + (L - 1) * G * H, L * G * H


def prepare(case, seed):
    """What a program that calls the library holds: inputs, parameters, states, upstream gradients (distributions of the
    shipped workloads), and the output, reserve and workspace buffers it allocated once for the shape."""
    L, T, B, I, H, G, nW, nR = _sizes(case)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    rnd = lambda *s: torch.randn(*s, device=dev, generator=g, dtype=torch.float32)  # noqa: E731
    uni = lambda n, a: (torch.rand(n, device=dev, generator=g, dtype=torch.float32) * 2 - 1) * a  # noqa: E731
    out = lambda *s: torch.empty(*s, device=dev, dtype=torch.float32)  # noqa: E731
    lstm = case["cell"] == "lstm"
    s = {"case": dict(case), "dims": (L, T, B, I, H)}
    s["x"], s["W"], s["R"], s["b"] = rnd(T, B, I), uni(nW, H ** -0.5), uni(nR, H ** -0.5), uni(L * G, 0.1)
    s["h0"], s["c0"] = rnd(L, B, H) * 0.1, rnd(L, B, H) * 0.1
    s["y"], s["hT"], s["cT"] = out(T, B, H), out(L, B, H), out(L, B, H)
    if lstm:
        rb, wb = lib.lstm_reserve_bytes(L, T, B, I, H), lib.lstm_workspace_bytes(L, T, B, I, H)
    else:
        s["code"] = lib.RNN_CELLS[case["cell"]]
        rb, wb = lib.rnn_reserve_bytes(s["code"], L, T, B, I, H), lib.rnn_workspace_bytes(s["code"], L, T, B, I, H)
    s["ws"], s["wb"], s["res"] = torch.empty(wb, dtype=torch.uint8, device=dev), wb, None
    # (rnn_forward keeps a reserve in every call)
    if case["train"] or not lstm:
        s["res"] = torch.empty(rb, dtype=torch.uint8, device=dev)
    if case["train"]:
        s["dy"] = rnd(T, B, H)
        s["dx"], s["dh0"], s["dc0"] = out(T, B, I), out(L, B, H), out(L, B, H)
        s["dW"], s["dR"], s["db"] = out(nW), out(nR), out(L * G)
    return s


def run(s):
    d = s["dims"]
    if s["case"]["cell"] == "lstm":
        lib.check(lib.lstm_forward(*d, s["x"], s["h0"], s["c0"], s["W"], s["R"], s["b"], s["y"], s["hT"], s["cT"], s["res"], s["ws"],
                                   s["wb"]), "lstm_forward")
        if s["case"]["train"]:
            lib.check(lib.lstm_backward(*d, s["x"], s["h0"], s["c0"], s["W"], s["R"], s["res"], s["dy"], None, None, s["dx"], s["dh0"],
                                        s["dc0"], s["dW"], s["dR"], s["db"], s["ws"], s["wb"]), "lstm_backward")
        names = ("y", "hT", "cT", "dx", "dh0", "dc0", "dW", "dR", "db")
        return {k: s[k] for k in (names if s["case"]["train"] else names[:3])}
    lib.check(lib.rnn_forward(s["code"], *d, s["x"], s["h0"], s["W"], s["R"], s["b"], s["y"], s["hT"], s["res"], s["ws"], s["wb"]),
              "rnn_forward")
    if s["case"]["train"]:
        lib.check(lib.rnn_backward(s["code"], *d, s["x"], s["h0"], s["W"], s["R"], s["res"], s["dy"], None, s["dx"], s["dh0"], s["dW"],
                                   s["dR"], s["db"], s["ws"], s["wb"]), "rnn_backward")
    names = ("y", "hT", "dx", "dh0", "dW", "dR", "db")
    return {k: s[k] for k in (names if s["case"]["train"] else names[:2])}


def work(case):
    """Every argument read once and every result written once; the products of each pass (forward; backward: gradients
    of the data, gradients of the weights)."""
    L, T, B, I, H, G, nW, nR = _sizes(case)
    states = (2 if case["cell"] == "lstm" else 1) * L * B * H
    params = nW + nR + L * G
    f = T * B * I + states + params + T * B * H + states
    flops = 2.0 * (nW + nR) * T * B
    if not case["train"]:
        return {"bytes": 4.0 * f, "flops": flops}
    # backward: x, states, weights, y's upstream gradient in; dx, state and parameter gradients out
    b = T * B * I + states + nW + nR + T * B * H + T * B * I + states + params
    return {"bytes": 4.0 * (f + b), "flops": 3.0 * flops}


def tolerance(case):
    """fp32 sums of up to 4H (or T*B) terms, carried through the steps."""
    return {"rel": 1e-5}


def exact(case, seed):
    """The same pass in float64, written out from the cells' equations."""
    if case["L"] * case["T"] > 2000:
        return None
    L, T, B, I, H, G, nW, nR = _sizes(case)
    s = prepare(case, seed)
    D = lambda k: s[k].double()  # noqa: E731
    cell = case["cell"]
    W = [D("W")[: G * I].view(G, I)] + list(D("W")[G * I:].view(L - 1, G, H)) if L > 1 else [D("W").view(G, I)]
    R, b = D("R").view(L, G, H), D("b").view(L, G)
    h0, c0 = D("h0"), D("c0")
    inp, saved = D("x"), []
    hT, cT = torch.empty_like(h0), torch.empty_like(c0)
    new = lambda *sh: torch.empty(*sh, dtype=torch.float64, device=inp.device)  # noqa: E731
    for l in range(L):
        P = (inp.reshape(T * B, -1) @ W[l].t()).view(T, B, G) + b[l]
        h, c = h0[l], c0[l]
        hs, cs, act, q3 = new(T, B, H), new(T, B, H), new(T, B, G), new(T, B, H)
        for t in range(T):
            Q = h @ R[l].t()
            if cell == "lstm":
                a = P[t] + Q
                sg, n = torch.sigmoid(a[:, : 3 * H]), torch.tanh(a[:, 3 * H:])
                c = sg[:, H: 2 * H] * c + sg[:, :H] * n
                h = sg[:, 2 * H:] * torch.tanh(c)
                act[t, :, : 3 * H], act[t, :, 3 * H:], cs[t] = sg, n, c
            elif cell == "gru":
                sg = torch.sigmoid(P[t, :, : 2 * H] + Q[:, : 2 * H])
                q3[t] = Q[:, 2 * H:]
                n = torch.tanh(P[t, :, 2 * H:] + sg[:, :H] * q3[t])
                h = (1 - sg[:, H:]) * n + sg[:, H:] * h
                act[t, :, : 2 * H], act[t, :, 2 * H:] = sg, n
            else:
                h = torch.tanh(P[t] + Q)
            hs[t] = h
        saved.append((inp, hs, cs, act, q3))
        hT[l], cT[l], inp = h, c, hs
    res = {"y": inp, "hT": hT}
    if cell == "lstm":
        res["cT"] = cT
    if not case["train"]:
        return res
    dW, dR, db = [None] * L, torch.empty_like(R), torch.empty_like(b)
    dh0, dc0, dout = torch.empty_like(h0), torch.empty_like(c0), D("dy")
    for l in reversed(range(L)):
        inp, hs, cs, act, q3 = saved[l]
        dA, dQ = new(T, B, G), new(T, B, G)  # gradients of W x + b and of R h
        dh, dc = torch.zeros_like(h0[l]), torch.zeros_like(h0[l])
        for t in reversed(range(T)):
            hp, cp = (hs[t - 1], cs[t - 1]) if t else (h0[l], c0[l])
            dh = dh + dout[t]
            if cell == "lstm":
                i, f, o, n = act[t].view(B, 4, H).unbind(1)
                tc = torch.tanh(cs[t])
                dc = dc + dh * o * (1 - tc * tc)
                dA[t] = torch.cat((dc * n * i * (1 - i), dc * cp * f * (1 - f), dh * tc * o * (1 - o), dc * i * (1 - n * n)), 1)
                dQ[t] = dA[t]
                dc, dh = dc * f, dA[t] @ R[l]
            elif cell == "gru":
                r, z, n = act[t].view(B, 3, H).unbind(1)
                dn = dh * (1 - z) * (1 - n * n)
                dr, dz = dn * q3[t] * r * (1 - r), dh * (hp - n) * z * (1 - z)
                dA[t], dQ[t] = torch.cat((dr, dz, dn), 1), torch.cat((dr, dz, dn * r), 1)
                dh = dh * z + dQ[t] @ R[l]
            else:
                dA[t] = dh * (1 - hs[t] * hs[t])
                dQ[t] = dA[t]
                dh = dA[t] @ R[l]
        dh0[l], dc0[l] = dh, dc
        flat = dA.view(T * B, G)
        dW[l] = (flat.t() @ inp.reshape(T * B, -1)).reshape(-1)
        dR[l] = dQ.view(T * B, G).t() @ torch.cat((h0[l][None], hs[:-1])).reshape(T * B, H)
        db[l] = flat.sum(0)
        dout = (flat @ W[l]).view(T, B, -1)
    res.update(dx=dout, dh0=dh0, dW=torch.cat(dW), dR=dR.reshape(-1), db=db.reshape(-1))
    if cell == "lstm":
        res["dc0"] = dc0
    return res
