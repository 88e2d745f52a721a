"""GPU parity of the kernels that run fp32 products on the fp16 matrix cores (factors split in two), where the split or its scaling
can go wrong: remainders, weights far from one, activations far from one, zero layers."""
import numpy as np
import pytest

import oracle
from paper_2309_12252_amd import deer, inputs
from helpers import DEV, TOL_ABS, dev, host, oracle_eval
from test_gpu_ode import check, check_grad

pytestmark = pytest.mark.gpu


def layers(w):
    """views of theta: (W_l, b_l) of every layer"""
    out, at = [], 0
    sizes = [w.n] + [w.mlp_width] * w.mlp_hidden_layers + [w.n]
    for k, m in zip(sizes[:-1], sizes[1:]):
        out.append((w.theta[at:at + m * k], w.theta[at + m * k:at + m * k + m]))
        at += m * k + m
    assert at == w.theta.size
    return out


def plain(w):
    pass


def far_scales(w):
    # a first layer that saturates, a second one below the smallest scale there is; (tanh's own absolute error must not be scaled up)
    l = layers(w)
    l[0][0][:] *= 64.0
    l[1][0][:] *= 2.0 ** -110


def large_activations(w):
    l = layers(w)
    l[0][1][:] += 700.0
    l[1][0][:] /= 256.0


def zero_layer(w):
    layers(w)[1][0][:] = 0.0


def faint_layer(w):
    # softplus units of about 2^-23 in front of weights of about 2^-100: what such a layer adds is its bias, large or zero
    l = layers(w)
    l[0][0][:] *= np.float32(0.1)
    l[0][1][:] = -15.5
    l[1][0][:] *= 2.0 ** -100
    l[1][1][0::3], l[1][1][1::3] = 0.0, 20.0


CASES = [(width, nhid, act, plain) for width in (32, 64) for nhid, act in
         ((1, inputs.ACT_SOFTPLUS), (2, inputs.ACT_SOFTPLUS), (3, inputs.ACT_TANH), (4, inputs.ACT_SOFTPLUS), (5, inputs.ACT_TANH))]
CASES += [(64, 4, inputs.ACT_TANH, far_scales), (32, 3, inputs.ACT_TANH, far_scales), (64, 5, inputs.ACT_SOFTPLUS, large_activations),
          (32, 2, inputs.ACT_SOFTPLUS, large_activations), (64, 3, inputs.ACT_TANH, zero_layer), (32, 5, inputs.ACT_SOFTPLUS, zero_layer),
          (64, 2, inputs.ACT_SOFTPLUS, faint_layer), (64, 5, inputs.ACT_SOFTPLUS, faint_layer), (32, 3, inputs.ACT_SOFTPLUS, faint_layer)]


@pytest.mark.parametrize("width,nhid,act,change", CASES)
def test_field(width, nhid, act, change):
    # (3 x 6,001 points: more than one sixteen of them to a SIMD, the last sixteen not full)
    for B, T in ((1, 3), (2, 37)) + (((3, 6001),) if change is plain else ()):
        w = inputs.mlp_ode_workload("split_w%d_L%d" % (width, nhid), 700 + width + nhid + B, B=B, T=T, n=8, width=width, nhid=nhid,
                                    t0=0.0, t1=1.0, tol=1e-4, act=act)
        change(w)
        check(w, deer.DEER_F32)
        # (the entries that multiply an activation of 700 are 700 times those of one: so is their rounding)
        check_grad(w, deer.DEER_F32, bar_theta=700 * TOL_ABS[deer.DEER_F32] if change is large_activations else None)


@pytest.mark.parametrize("width,nhid,act", [(32, 2, inputs.ACT_TANH), (64, 2, inputs.ACT_TANH), (64, 3, inputs.ACT_SOFTPLUS)])
@pytest.mark.parametrize("B,T", [(1, 2), (7, 2), (1, 16), (1, 17), (2, 15), (5, 31), (3, 7000)])
def test_field_of_few_points_and_many(width, nhid, act, B, T):
    # the two-layer field at widths 32 and 64: fewer points than sixteen, exactly as many, one more, more than one block of them to a SIMD
    w = inputs.mlp_ode_workload("points_w%d_T%d" % (width, T), 820 + width + T, B=B, T=T, n=8, width=width, nhid=nhid, t0=0.0, t1=1.5, tol=1e-4, act=act)
    check(w, deer.DEER_F32)


@pytest.mark.parametrize("width,nhid", [(32, 2), (64, 2), (32, 1)])
def test_field_on_a_coarse_grid(width, nhid):
    # few points over a long span: the series is evaluated on scaled matrices, by other numbers of terms and doublings from interval to interval
    w = inputs.mlp_ode_workload("coarse_w%d" % width, 77 + width, B=3, T=12, n=8, width=width, nhid=nhid, t0=0.0, t1=6.0, tol=1e-4)
    w.theta = (w.theta * 2.0).astype(np.float32)
    check(w, deer.DEER_F32)


# Reduction by chunks: Jacobians whose entries lie beyond the range of fp16 (the chunk is reduced again with fp32 products), products that leave it within a
# chunk, ordinary ones, and ones next to nothing (whose digits the next test looks at).  One step from zero, every position against max(1, its own size): fp32 rounding
# grows by the conditioning of up to eleven products (1e-7 each, some hundred times that where terms cancel).
@pytest.mark.parametrize("n", [16, 32, 64, 27, 50])
@pytest.mark.parametrize("scale,T", [(3.0e6, 5), (40.0, 11), (1.0, 300), (2.0 ** -9, 300)])
@pytest.mark.parametrize("L", ["4", "8"])
def test_range_of_the_reduction(n, scale, T, L, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", L)
    d, B = 3, 3
    w = inputs.gru_workload("range", 640 + n, B=B, T=T, n=n, d=d)
    U = w.theta[3 * n * d:3 * n * d + 3 * n * n]
    U *= np.float32(scale)
    if scale < 1.0:
        w.theta[3 * n * d + 3 * n * n + n:][:n] = -7.0   # z = 1e-3: nothing but small entries
    want = oracle.deer_eval(oracle.make_cell(oracle.CELL_GRU, n, d), w.theta, w.x, w.y0, tol=w.tol, max_iter=1, nthreads=8)[0]
    ctx = deer.context_for(w, device=DEV)
    try:
        y = host(ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=w.tol, max_iter=1)[0])
    finally:
        ctx.close()
    off = np.abs(y - want).max(axis=-1) / np.maximum(1.0, np.abs(want).max(axis=-1))
    print(n, scale, L, "%.1e, iterate up to %.1e" % (off.max(), np.abs(want).max()), flush=True)
    assert off.max() <= 1e-4


# One column of the running product leaves the range of fp16, in lanes of one wavefront that are not its first: row i of J has entries of some 1e4 and no other row
# reads channel i.  All chunks are reduced again, those of the other wavefronts (n = 64: a workgroup's four share a unit) too.
@pytest.mark.parametrize("n,i", [(16, 5), (32, 21), (64, 5), (64, 37), (64, 63)])
def test_one_column_leaves_the_range(n, i, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", "8")
    d, B, T = 3, 3, 300
    w = inputs.gru_workload("one_column", 660 + n + i, B=B, T=T, n=n, d=d)
    U = w.theta[3 * n * d:3 * n * d + 3 * n * n].reshape(3, n, n)
    U[:, :, i] = 0.0
    U[2, i] *= np.float32(3e5)
    cell = oracle.make_cell(oracle.CELL_GRU, n, d)
    want = oracle.deer_eval(cell, w.theta, w.x, w.y0, tol=w.tol, max_iter=1, nthreads=8)[0]
    assert np.abs(want[..., i]).max() > 1e4 and np.abs(np.delete(want, i, axis=-1)).max() < 10.0
    ctx = deer.context_for(w, device=DEV)
    try:
        first, last = [host(ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=w.tol, max_iter=m)[0]) for m in (1, 12)]
    finally:
        ctx.close()
    # Entry by entry, against the largest in its place, with the weights of row i 1e5 times the others.  A step rounds about eight times (2^-24 each), what is
    # older than eight steps has faded; four times the root of their sum.  (The solution: without channel i, which is a sign of rounded sums.)
    bound = 4.0 * np.sqrt(8.0 * 8.0) * 2.0 ** -24
    off = (np.abs(first - want) / np.maximum(1.0, np.abs(want).max(axis=(0, 1)))).max()
    rest = np.abs(np.delete(last - oracle.seq_eval(cell, w.theta, w.x, w.y0, nthreads=8), i, axis=-1)).max()
    print(n, i, "%.1e %.1e of %.1e" % (off, rest, bound), flush=True)
    assert off <= bound and rest <= bound


# What the field leaves out at many points in a row adds up along a trajectory, and the rounding of the stored states, twice as large, hides it: so the mean error over the last
# fifth, 24 solves.  Sums rounded to fp32 term by term leave 1.46e-8 and 1.00e-8 of the states there; a quarter more is the spread of 24 solves
# (rounding 2^-24 of sums that scatter, on a path of length one).  Sums whose rounding repeats from point to point leave 2.2e-8 and 1.8e-8.
@pytest.mark.parametrize("nhid,fp32", [(2, 1.46e-8), (3, 1.00e-8)])
def test_field_does_not_drift(nhid, fp32):
    off = []
    for seed in range(24):
        w = inputs.mlp_ode_workload("drift", 3000 + seed, B=4, T=5000, n=8, width=32, nhid=nhid, t0=0.0, t1=10.0, tol=1e-4, act=inputs.ACT_SOFTPLUS)
        ctx = deer.context_for(w, device=DEV)
        try:
            th, y0 = dev(w.theta, 0), dev(w.y0, 0)
            y = ctx.eval(th, None, y0, tol=w.tol, max_iter=w.max_iter)[0]
            y = host(ctx.eval(th, None, y0, y_guess=y, tol=0.0, max_iter=3)[0])
        finally:
            ctx.close()
        want = oracle_eval(w, tol=1e-10, guess=y)[0]
        e = (y - want)[:, -1000:].mean(axis=1)
        off.append(np.linalg.norm(e) / np.linalg.norm(np.sqrt((want[:, -1000:] ** 2).mean(axis=1))))
    rms = np.sqrt(np.mean(np.square(off)))
    print(nhid, "%.2e of %.2e" % (rms, 1.25 * fp32), flush=True)
    assert rms <= 1.25 * fp32


# The same at single positions, another one in every sequence: what was reduced before it is kept, its chunk and those behind it are reduced again.  The reset gate lets
# the large weights of row i through where the first input says so.
@pytest.mark.parametrize("kind,n", [("gru", 16), ("gru", 32), ("gru", 64), ("lstm", 16)])
@pytest.mark.parametrize("L", ["4", "16", "24", "64"])
def test_one_position_leaves_the_range(kind, n, L, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", L)
    d, B, T, i = 3, 24, 1100, 5
    gates = 3 if kind == "gru" else 4
    make = inputs.gru_workload if kind == "gru" else inputs.lstm_workload
    w = make("one_position", 680 + n, B, T, n, d)
    W, U = w.theta[:gates * n * d].reshape(gates, n, d), w.theta[gates * n * d:][:gates * n * n].reshape(gates, n, n)
    bias = w.theta[gates * n * d + gates * n * n:].reshape(-1, n)
    gate = 0   # GRU: reset, in front of the candidate's U; LSTM: input, in front of g
    W[gate, i], bias[gate, i] = 0.0, -40.0
    W[gate, i, 0] = 80.0
    U[:, :, i] = 0.0
    U[gate, i] = 0.0
    U[2, i] *= np.float32(3e5)
    w.x[:, :, 0] = 0.0
    at = np.random.default_rng(9).integers(0, T, size=B)
    at[:4] = 0, 1, T // 2, T - 1
    w.x[np.arange(B), at, 0] = 1.0
    cell = oracle.make_cell(oracle.CELL_GRU if kind == "gru" else oracle.CELL_LSTM, n if kind == "gru" else 2 * n, d)
    want = oracle.deer_eval(cell, w.theta, w.x, w.y0, tol=w.tol, max_iter=1, nthreads=8)[0]
    ctx = deer.context_for(w, device=DEV)
    try:
        y = host(ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=w.tol, max_iter=1)[0])
    finally:
        ctx.close()
    size = np.abs(want).max(axis=(0, 1))
    assert size.max() > 1e4
    # (the bound of the whole column above; the large entries' rounding reaches the rest through the state's second half only, whose place is large too)
    bound = 4.0 * np.sqrt(8.0 * 8.0) * 2.0 ** -24
    off = (np.abs(y - want) / np.maximum(1.0, size)).max()
    print(kind, n, L, "%.1e of %.1e, up to %.1e" % (off, bound, size.max()), flush=True)
    assert off <= bound


# Products that fade, against their own size.  Without inputs and biases (but the one that keeps the old state) the cell is zero at zero, so one step from zero carries what y0 leaves at
# the first position through the chunks' maps alone, and every position is that times a product of Jacobians.
@pytest.mark.parametrize("kind,n,bias,T", [("gru", n, *b) for n in (16, 27, 32, 50, 64) for b in ((0.0, 150), (-1.0, 64), (-2.0, 40))] +
                         [("lstm", n, *b) for n in (12, 16) for b in ((1.0, 150), (0.0, 150))])
@pytest.mark.parametrize("L", ["4", "16", "32", "64"])
def test_products_that_fade(kind, n, bias, T, L, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", L)
    d, B = 3, 3
    w = (inputs.gru_workload if kind == "gru" else inputs.lstm_workload)("fade", 720 + n + T, B, T, n, d)
    gates, ch = (3, n) if kind == "gru" else (4, 2 * n)
    w.theta[:gates * n * d] = 0.0
    b = w.theta[gates * n * d + gates * n * n:].reshape(-1, n)
    b[:] = 0.0
    b[1] = bias
    w.y0 = (np.random.default_rng(n).standard_normal((B, ch)) * 0.5).astype(np.float32)
    cell = oracle.make_cell(oracle.CELL_GRU if kind == "gru" else oracle.CELL_LSTM, ch, d)
    want = oracle.deer_eval(cell, w.theta, w.x, w.y0, tol=w.tol, max_iter=1, nthreads=8)[0]
    ctx = deer.context_for(w, device=DEV)
    try:
        y = host(ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=w.tol, max_iter=1)[0])
    finally:
        ctx.close()
    size = np.linalg.norm(want, axis=-1)
    off = (np.linalg.norm(y - want, axis=-1) / size).max()
    # fp32: a step rounds about eight times, as in the gradient's test; the Jacobian is the same at every position here, so what its gate and its entry round (twice 2^-24) is
    # the same too and grows by the number of positions.  Split: between two looks a column falls by 2^k from at least 2^3, and an entry of it is off by 2^-25; as
    # many entries as channels, four times that for the products on the way.
    k = np.log2((size[:, :-16] / size[:, 16:]).max())
    bound = (4.0 * np.sqrt(8.0 * (T + 1)) + 2.0 * (T + 1)) * 2.0 ** -24 + 4.0 * np.sqrt(ch) * 2.0 ** (k - 28)
    print(kind, n, bias, L, "%.1e of %.1e, down to %.1e, 2^%.0f in sixteen positions" % (off, bound, size.min(), -k), flush=True)
    assert size.min() > 1e-34 and bound < 0.02 and off <= bound
