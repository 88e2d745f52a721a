"""GPU parity of the gradient of a loss on the last state only, by chunks: the cotangent fades on its way back over several chunks, and what is left of it at
each position, and in dL/dy0, is compared with the fp64 oracle relative to its own size."""
import numpy as np
import pytest

import oracle
from paper_2309_12252_amd import deer, inputs
from helpers import DEV, dev, host

pytestmark = pytest.mark.gpu


# bias: what is added to the gate that keeps the old state (GRU: z, LSTM: f; LEM: taken from both time scales, whose rest 1 - s keeps it), so that a step keeps about
# 0.5, 0.27 or 0.12 of the state.  A chunk's map is a product of up to 64 Jacobians.
@pytest.mark.parametrize("kind,n", [("gru", 16), ("gru", 27), ("gru", 32), ("gru", 50), ("gru", 64), ("lstm", 8), ("lstm", 12), ("lstm", 16), ("lem", 8), ("lem", 12), ("lem", 16)])
@pytest.mark.parametrize("bias,T", [(0.0, 150), (-1.0, 64), (-2.0, 40)])
@pytest.mark.parametrize("L", ["16", "32", "64"])
def test_cotangent_at_the_last_position(kind, n, bias, T, L, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", L)
    d, B = 6, 3
    make = {"gru": inputs.gru_workload, "lstm": inputs.lstm_workload, "lem": inputs.lem_workload}[kind]
    w = make("fading", 5200 + n + T, B, T, n, d)
    gates = 3 if kind == "gru" else 4
    b = w.theta[gates * n * d + gates * n * n:][:gates * n].reshape(gates, n)
    if kind == "lem":
        b[:2] -= np.float32(bias)
    else:
        b[1] += np.float32(bias)
    ch = n if kind == "gru" else 2 * n
    w.y0 = (np.random.default_rng(n).standard_normal((B, ch)) * 0.5).astype(np.float32)
    c = oracle.make_cell({"gru": oracle.CELL_GRU, "lstm": oracle.CELL_LSTM, "lem": oracle.CELL_LEM}[kind], ch, d, **({"dt": w.t1} if kind == "lem" else {}))
    y = oracle.seq_eval(c, w.theta, w.x, w.y0, nthreads=8).astype(np.float32).astype(np.float64)
    g = np.zeros_like(y)
    g[:, -1] = np.random.default_rng(1).standard_normal((B, ch)).astype(np.float32)
    want = (oracle.gru_grad(n, d, w.theta, w.x, w.y0, y, g) if kind == "gru" else oracle.rnn_grad(c, w.theta, w.x, w.y0, y, g))
    ctx = deer.context_for(w, device=DEV)
    try:
        got = [host(t) for t in ctx.grad(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), dev(y, 0), dev(g, 0))]
    finally:
        ctx.close()
    # A step rounds about eight times on the way of an entry (gates, factors, the sum of the product): 2^-24 each, independent, and four times that for
    # what the gates' own functions and terms that cancel add; blocks of eight positions of dL/dx, which are nowhere near the smallest fp32 numbers.
    bound = 4.0 * np.sqrt(8.0 * (T + 1)) * 2.0 ** -24
    pairs = [("dy0", got[2], want[2])] + [("dx %d" % t, got[1][:, t:t + 8], want[1][:, t:t + 8]) for t in range(0, T - 8, 8)]
    worst = max((np.linalg.norm(a - b) / np.linalg.norm(b), name, np.linalg.norm(b)) for name, a, b in pairs)
    print(kind, n, bias, L, "%.2e (%s, norm %.1e) of %.2e" % (worst + (bound,)), flush=True)
    assert np.linalg.norm(want[2]) > 1e-34
    assert worst[0] <= bound
