"""GPU parity of the GRU step and dual scan by chunks (fp32, n = 16, 32, 64) at the edges of chunks, groups of sixteen chunks and blocks
of sixteen positions: trajectory, iteration count and gradients against the fp64 oracle, plain max-abs at 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_12252_amd import deer, inputs
from helpers import DEV, dev, host, gpu_eval, oracle_cell, oracle_eval

pytestmark = pytest.mark.gpu

# (chunk length, B, T): one position, a single ragged chunk, group boundaries (16 chunks) minus / plus one position, several
# groups with the last one ragged, chunks that are no multiple of the sixteen-position block, few and many groups
SHAPES = [(4, 1, 1), (4, 2, 3), (4, 1, 64), (4, 3, 65), (8, 2, 127), (8, 1, 129), (20, 2, 1000), (12, 3, 1543), (36, 1, 2049), (100, 2, 3300)]


@pytest.mark.parametrize("n,d", [(16, 1), (16, 6), (16, 16), (32, 4), (32, 8), (32, 13), (24, 3), (64, 3), (64, 8), (64, 16), (50, 5)])
def test_step_and_dual_by_chunks(n, d, monkeypatch):
    for k, (L, B, T) in enumerate(SHAPES):
        monkeypatch.setenv("DEER_CHUNK_L", str(L))
        monkeypatch.setenv("DEER_CHUNK_UNIT", str((4, 8, 16)[k % 3]))
        w = inputs.gru_workload("chunk_n%d_L%d_T%d" % (n, L, T), 1300 + 20 * n + k, B=B, T=T, n=n, d=d)
        w.y0 = np.random.default_rng(k).standard_normal((B, n)).astype(np.float32)
        print(w.name, B, d, flush=True)
        yo, ito, _, _ = oracle_eval(w)
        yg, itg, _, conv, st = gpu_eval(w)
        assert st == deer.DEER_OK and conv and abs(itg - ito) <= 1, (w.name, itg, ito)
        assert np.abs(yg - yo).max() <= 1e-4, (w.name, np.abs(yg - yo).max())
        y2, _, _, _, _ = gpu_eval(w, max_iter=2)   # an iterate far from the solution
        assert np.abs(y2 - oracle_eval(w, max_iter=2)[0]).max() <= 1e-4, w.name
        g = (np.random.default_rng(k + 1).standard_normal((B, T, n)) / np.sqrt(T)).astype(np.float32).astype(np.float64)
        y = oracle.seq_eval(oracle_cell(w), w.theta, w.x, w.y0, nthreads=8)
        want = oracle.gru_grad(w.n, w.d, w.theta, w.x, w.y0, y, g)
        ctx = deer.context_for(w, device=DEV)
        try:
            got = ctx.grad(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), dev(y, 0), dev(g, 0))
        finally:
            ctx.close()
        for name, a, b in zip(("dtheta", "dx", "dy0"), got, want):
            assert np.abs(host(a) - b).max() <= 1e-4, (w.name, name, np.abs(host(a) - b).max())


@pytest.mark.parametrize("cell", [oracle.CELL_LSTM, oracle.CELL_LEM], ids=["lstm", "lem"])
@pytest.mark.parametrize("u,d", [(1, 2), (4, 8), (6, 3), (8, 4), (8, 8), (9, 1), (12, 6), (15, 5), (16, 8)])
def test_two_part_cells_by_chunks(cell, u, d, monkeypatch):
    # 1 to 8 units share one 16 x 16 block, 9 to 16 take a block per part; unit counts that are no multiple of four take scalar accesses
    for k, (L, B, T) in enumerate(SHAPES):
        monkeypatch.setenv("DEER_CHUNK_L", str(L))
        monkeypatch.setenv("DEER_CHUNK_UNIT", str((4, 8, 16)[k % 3]))
        make = inputs.lstm_workload if cell == oracle.CELL_LSTM else inputs.lem_workload
        # (one input of the LEM is drawn with another seed: with the plain one the oracle's iterates reach 1e16 before they converge after 22 iterations,
        # and how many it takes depends on every rounding)
        far = cell == oracle.CELL_LEM and (u, d, T) == (9, 1, 1543)
        w = make("chunk_u%d_L%d_T%d" % (u, L, T), 1700 + 20 * u + k + (1000 if far else 0), B=B, T=T, units=u, d=d)
        w.y0 = (np.random.default_rng(k).standard_normal((B, 2 * u)) * 0.5).astype(np.float32)
        print(cell, w.name, B, d, flush=True)
        c = oracle.make_cell(cell, 2 * u, d, **({} if cell == oracle.CELL_LSTM else {"dt": w.t1}))
        ctx = deer.context_for(w, device=DEV)
        try:
            th, x, y0 = dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0)
            yo, ito, erro, _ = oracle.deer_eval(c, w.theta, w.x, w.y0, tol=w.tol, max_iter=w.max_iter, nthreads=8)
            y, it, _, conv, st = ctx.eval(th, x, y0, tol=w.tol, max_iter=w.max_iter)
            assert st == deer.DEER_OK and conv and erro <= w.tol and abs(it - ito) <= 1, (w.name, it, ito)
            assert np.abs(host(y) - yo).max() <= 1e-4, (w.name, np.abs(host(y) - yo).max())
            # an iterate far from the solution: every position against its own size
            yo = oracle.deer_eval(c, w.theta, w.x, w.y0, tol=w.tol, max_iter=2, nthreads=8)[0]
            off = np.abs(host(ctx.eval(th, x, y0, tol=w.tol, max_iter=2)[0]) - yo).max(axis=-1)
            assert (off <= 1e-4 * np.maximum(1.0, np.abs(yo).max(axis=-1))).all(), (w.name, off.max())
            ys = oracle.seq_eval(c, w.theta, w.x, w.y0, nthreads=8)
            g = (np.random.default_rng(k + 1).standard_normal(ys.shape) / np.sqrt(T)).astype(np.float32).astype(np.float64)
            want = oracle.rnn_grad(c, w.theta, w.x, w.y0, ys, g)
            got = ctx.grad(th, x, y0, dev(ys, 0), dev(g, 0))
        finally:
            ctx.close()
        for name, a, b in zip(("dtheta", "dx", "dy0"), got, want):
            assert np.abs(host(a) - b).max() <= 1e-4, (w.name, name, np.abs(host(a) - b).max())


def _against_oracle(ctx, w, oracle_solve, oracle_sequential, oracle_gradient):
    th, x, y0 = dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0)
    for max_iter in (w.max_iter, 2):   # the solution and an iterate far from it
        yo, ito, _, _ = oracle_solve(max_iter)
        y, it, _, _, st = ctx.eval(th, x, y0, tol=w.tol, max_iter=max_iter)
        assert st == deer.DEER_OK and abs(it - ito) <= 1, (w.name, it, ito)
        assert np.abs(host(y) - yo).max() <= 1e-4, (w.name, max_iter, np.abs(host(y) - yo).max())
    ys = oracle_sequential()
    g = (np.random.default_rng(1).standard_normal(ys.shape) / np.sqrt(w.T)).astype(np.float32).astype(np.float64)
    got = ctx.grad(th, x, y0, dev(ys, 0), dev(g, 0))
    for name, a, b in zip(("dtheta", "dx", "dy0"), got, oracle_gradient(ys, g)):
        assert np.abs(host(a).reshape(-1) - b.reshape(-1)).max() <= 1e-4, (w.name, name, np.abs(host(a).reshape(-1) - b.reshape(-1)).max())


@pytest.mark.parametrize("n,d", [(8, 1), (8, 4), (8, 8), (5, 3), (7, 6)])
def test_eight_channels_by_chunks(n, d, monkeypatch):
    for k, (L, B, T) in enumerate(SHAPES):
        monkeypatch.setenv("DEER_CHUNK_L", str(L))
        w = inputs.gru_workload("chunk_n%d_L%d_T%d" % (n, L, T), 2100 + 20 * n + k, B=B, T=T, n=n, d=d)
        w.y0 = np.random.default_rng(k).standard_normal((B, n)).astype(np.float32)
        print(w.name, B, d, flush=True)
        ctx = deer.context_for(w, device=DEV)
        try:
            _against_oracle(ctx, w, lambda m: oracle_eval(w, max_iter=m), lambda: oracle.seq_eval(oracle_cell(w), w.theta, w.x, w.y0, nthreads=8),
                            lambda ys, g: oracle.gru_grad(w.n, w.d, w.theta, w.x, w.y0, ys, g))
        finally:
            ctx.close()


# recurrences of 1, 2, 4, 8 and more than 16 chunks in one launch, fewer steps than the largest stride, groups of sixteen columns that
# several batch entries share, one head, head counts that are no multiple of the levels
@pytest.mark.parametrize("n,d", [(8, 1), (8, 4), (8, 7), (8, 8)])
@pytest.mark.parametrize("L,B,T,H,K", [(4, 1, 1, 3, 2), (4, 2, 5, 6, 4), (8, 3, 300, 4, 3), (16, 1, 131, 8, 8), (12, 2, 1030, 11, 8), (32, 5, 333, 1, 4),
                                       (64, 2, 700, 5, 2), (4, 1, 1543, 3, 3)])
def test_heads_by_chunks(n, d, L, B, T, H, K, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", str(L))
    w = inputs.mh_gru_workload("chunk_mh_n%d_H%d_K%d_T%d" % (n, H, K, T), 2500 + T + 40 * n + d, B=B, T=T, n=n, d=d, H=H, K=K)
    w.y0 = np.random.default_rng(3).standard_normal((B, H, n)).astype(np.float32)
    ctx = deer.context_for(w, device=DEV)
    try:
        _against_oracle(ctx, w, lambda m: oracle.mh_deer_eval(n, d, H, K, w.theta, w.x, w.y0, tol=w.tol, max_iter=m, nthreads=8),
                        lambda: oracle.mh_seq_eval(n, d, H, K, w.theta, w.x, w.y0, nthreads=8),
                        lambda ys, g: oracle.mh_gru_grad(n, d, H, K, w.theta, w.x, w.y0, ys, g))
    finally:
        ctx.close()


# the gradient alone (no dL/dx, no dL/dy0) is the same sum in the same order, and eight channels need no more than the alignment of a scalar
@pytest.mark.parametrize("kind,n", [("gru", 8), ("gru", 16), ("gru", 64), ("heads", 8), ("lstm", 8), ("lem", 12)])
def test_parameter_gradient_alone_and_scalar_alignment(kind, n, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", "12")
    B, T, d = 3, 413, 5
    if kind == "heads":
        w = inputs.mh_gru_workload("chunk_alone_mh", 71, B=B, T=T, n=n, d=d, H=3, K=3)
    elif kind == "gru":
        w = inputs.gru_workload("chunk_alone_n%d" % n, 72 + n, B=B, T=T, n=n, d=d)
    else:
        w = (inputs.lstm_workload if kind == "lstm" else inputs.lem_workload)("chunk_alone_" + kind, 73, B=B, T=T, units=n, d=d)

    def at_odd_scalar(t):   # the same values one scalar behind an aligned address
        flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
        flat[1:] = t.reshape(-1)
        return flat[1:].reshape(t.shape)

    ctx = deer.context_for(w, device=DEV)
    try:
        th, x, y0 = dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0)
        y = ctx.eval(th, x, y0, tol=w.tol, max_iter=w.max_iter)[0]
        g = dev((np.random.default_rng(2).standard_normal(tuple(y.shape)) / T).astype(np.float32), 0)
        dth, dx, dy0 = ctx.grad(th, x, y0, y, g)
        alone = ctx.grad(th, x, y0, y, g, want_dx=False, want_dy0=False)
        assert alone[1] is None and alone[2] is None and torch.equal(alone[0], dth)
        if n == 8 and kind in ("gru", "heads"):
            odd = [at_odd_scalar(t) for t in (th, x, y0)]
            assert odd[0].data_ptr() % 8 == 4
            assert torch.equal(ctx.eval(*odd, tol=w.tol, max_iter=w.max_iter)[0], y)
            for a, b in zip(ctx.grad(*odd, at_odd_scalar(y), at_odd_scalar(g)), (dth, dx, dy0)):
                assert torch.equal(a, b)
    finally:
        ctx.close()


# Error against 64 bits: no larger than that of the scans, which sum about sixteen positions at a time.  Relative 2-norm, mean over three inputs; a tenth
# on top for the scatter of such a mean (dL/dtheta has 416 entries and more; dL/dy0 is compared where it has as many).
@pytest.mark.parametrize("kind,n,d,B,T,H,K", [("heads", 8, 8, 8, 1024, 32, 8), ("gru", 8, 5, 16, 12003, 0, 0), ("gru", 16, 6, 8, 9001, 0, 0), ("gru", 27, 9, 6, 9001, 0, 0),
                                              ("gru", 50, 7, 9, 4001, 0, 0), ("gru", 64, 16, 8, 4003, 0, 0),
                                              ("lstm", 8, 4, 8, 12000, 0, 0), ("lstm", 12, 3, 5, 7001, 0, 0), ("lem", 8, 3, 5, 7001, 0, 0), ("lem", 16, 6, 8, 9001, 0, 0)])
def test_gradient_error_no_larger_than_the_scans(kind, n, d, B, T, H, K, monkeypatch):
    cell = {"lstm": deer.DEER_CELL_LSTM, "lem": deer.DEER_CELL_LEM}.get(kind, deer.DEER_CELL_GRU)
    ch = 2 * n if kind in ("lstm", "lem") else n
    lead, state = ((B, T, H), (B, H, n)) if H else ((B, T), (B, ch))
    config = lambda dtype: deer.make_config(cell, dtype, B, T, n, d=d, t1=1.0 if kind == "lem" else 0.0, heads=H, stride_levels=K)
    by_scan = {"DEER_FUSED_L": "4"} if n == 8 and cell == deer.DEER_CELL_GRU else {"DEER_FUSED": "0", "DEER_VJP_MFMA": "1" if n <= 32 else "0"}
    err = {}
    for seed in range(3):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(900 + seed)
        normal = lambda *shape: torch.randn(*shape, generator=gen, device=DEV)
        theta = normal(deer.theta_count(config(deer.DEER_F32))) / np.sqrt(n)
        x, y0, g = normal(*lead, d), torch.zeros(*state, device=DEV), normal(*lead, ch) / (B * T)
        if n <= 32:
            ctx = deer.DeerContext(config(deer.DEER_F64), device=DEV)
            y = ctx.eval(theta.double(), x.double(), y0.double(), tol=1e-9, max_iter=50)[0]
            want = ctx.grad(theta.double(), x.double(), y0.double(), y, g.double())
            ctx.close()
        else:   # (state sizes above 32 run in fp32 only)
            h = [t.double().cpu().numpy() for t in (theta, x, y0, g)]
            y = oracle.seq_eval(oracle.make_cell(oracle.CELL_GRU, n, d), h[0], h[1], h[2], nthreads=8)
            want = [torch.from_numpy(a).to(DEV) for a in oracle.gru_grad(n, d, h[0], h[1], h[2], y, h[3])]
            y = torch.from_numpy(y).to(DEV)
        for route, knobs in (("chunks", {"DEER_CHUNK_L": "32"}), ("scans", by_scan)):
            with monkeypatch.context() as m:
                for k, v in knobs.items():
                    m.setenv(k, v)
                ctx = deer.DeerContext(config(deer.DEER_F32), device=DEV)
                got = ctx.grad(theta, x, y0, y.float(), g)
                ctx.close()
            for name, a, b in zip(("dtheta", "dx", "dy0"), got, want):
                err[route, name] = err.get((route, name), 0.0) + float((a.double() - b).norm() / b.norm()) / 3
    for name in ("dtheta", "dx") + (("dy0",) if y0.numel() >= 400 else ()):
        print(kind, n, name, "%.3g %.3g" % (err["chunks", name], err["scans", name]), flush=True)
        assert err["chunks", name] <= 1.1 * err["scans", name], (name, err)


# n = 64: the four wavefronts of a workgroup go through several blocks of sixteen positions each (512 workgroups: more than 8,192 positions),
# sequences start in later ones, with and without dL/dx and dL/dy0; chunk lengths by default
@pytest.mark.parametrize("n,d,B,T", [(64, 8, 5, 9973), (50, 7, 300, 61), (64, 16, 2, 20011)])
def test_parameter_sums_over_many_positions_at_64(n, d, B, T):
    w = inputs.gru_workload("many64", 3100 + n + T, B=B, T=T, n=n, d=d)
    w.y0 = np.random.default_rng(5).standard_normal((B, n)).astype(np.float32)
    ctx = deer.context_for(w, device=DEV)
    try:
        _against_oracle(ctx, w, lambda m: oracle_eval(w, max_iter=m), lambda: oracle.seq_eval(oracle_cell(w), w.theta, w.x, w.y0, nthreads=8),
                        lambda ys, g: oracle.gru_grad(w.n, w.d, w.theta, w.x, w.y0, ys, g))
        y = ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=w.tol, max_iter=w.max_iter)[0]
        g = dev((np.random.default_rng(2).standard_normal(tuple(y.shape)) / T).astype(np.float32), 0)
        run = lambda **kw: ctx.grad(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), y, g, **kw)
        whole, alone = run(), run(want_dx=False, want_dy0=False)
        assert torch.equal(whole[0], alone[0]) and torch.equal(run(want_dx=False)[2], whole[2]) and torch.equal(run(want_dy0=False)[1], whole[1])
    finally:
        ctx.close()


# Jacobians that expand where the correction is zero: no input over the first 2,000 steps and no bias, so the state stays at the origin, where a step
# multiplies by 1.5 to 1.9; then a signal that saturates the cell.  Chunks of 32 positions do not overflow, units and groups of sixteen of them do
# (1.5^512), and so would the product over all 2,000 steps.  The solve starts from the solution and the cotangent ends after ten steps, so nothing that
# is computed is large: the trajectory and the gradient are those of the oracle.
@pytest.mark.parametrize("kind,n", [("gru", 8), ("gru", 16), ("gru", 27), ("gru", 64), ("heads", 8), ("lstm", 8), ("lstm", 12), ("lem", 7), ("lem", 16)])
@pytest.mark.parametrize("unit", ["4", "16"])
def test_expanding_jacobians_and_no_correction(kind, n, unit, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", "32" if unit == "16" else "64")
    monkeypatch.setenv("DEER_CHUNK_UNIT", unit)
    rng = np.random.default_rng(17 + n)
    B, T, d, quiet, H, K = 2, 3001, 3, 2000, 3, 2
    gates = 3 if kind in ("gru", "heads") else 4
    cells = H if kind == "heads" else 1
    theta = []
    for _ in range(cells):
        W, U = rng.standard_normal((gates, n, d)), 0.1 * rng.standard_normal((gates, n, n)) / np.sqrt(n)
        for gate in (2, 3) if kind == "lem" else (2,):
            U[gate] += (2.0 if kind == "lem" else 4.0) * np.eye(n)
        theta += [W.ravel(), U.ravel(), np.zeros(4 * n)]
    ch = 2 * n if kind in ("lstm", "lem") else n
    lead = (B, T, H) if kind == "heads" else (B, T)
    x = rng.standard_normal(lead + (d,))
    x[:, :quiet] = 0.0
    y0 = np.zeros((B, H, n) if kind == "heads" else (B, ch))
    g = np.zeros(lead + (ch,))
    g[:, :10] = 1e-3 * rng.standard_normal(g[:, :10].shape)
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32).astype(np.float64)
    theta, x, g = f32(np.concatenate(theta)), f32(x), f32(g)
    if kind == "heads":
        solve = lambda th: oracle.mh_seq_eval(n, d, H, K, th, x, y0, nthreads=8)
        ys = solve(theta)
        want = oracle.mh_gru_grad(n, d, H, K, theta, x, y0, ys, g)
    else:
        c = oracle.make_cell({"gru": oracle.CELL_GRU, "lstm": oracle.CELL_LSTM, "lem": oracle.CELL_LEM}[kind], ch, d, **({"dt": 1.0} if kind == "lem" else {}))
        solve = lambda th: oracle.seq_eval(c, th, x, y0, nthreads=8)
        ys = solve(theta)
        want = oracle.gru_grad(n, d, theta, x, y0, ys, g) if kind == "gru" else oracle.rnn_grad(c, theta, x, y0, ys, g)
    assert np.abs(ys[:, :quiet]).max() == 0.0 and np.abs(ys[:, quiet + 200:]).max() > 0.5
    # where the signal sets in, a state near the origin carries every rounding along: what weights off by one in 2^24 change in the solution, times
    # eight for the products, the gates and the state that are rounded too (1e-4 where that is less)
    bound = max(1e-4, 8.0 * np.abs(solve(theta * (1.0 + 2.0 ** -24 * rng.choice([-1.0, 1.0], theta.shape))) - ys).max())
    cell = {"lstm": deer.DEER_CELL_LSTM, "lem": deer.DEER_CELL_LEM}.get(kind, deer.DEER_CELL_GRU)
    ctx = deer.DeerContext(deer.make_config(cell, deer.DEER_F32, B, T, n, d=d, t1=1.0 if kind == "lem" else 0.0, heads=H if kind == "heads" else 0,
                                            stride_levels=K if kind == "heads" else 0), device=DEV)
    try:
        th, xd, y0d = dev(theta, 0), dev(x, 0), dev(y0, 0)
        y, it, _, conv, st = ctx.eval(th, xd, y0d, y_guess=dev(ys, 0), tol=1e-4, max_iter=20)
        assert st == deer.DEER_OK and conv
        print(kind, n, "%.2e of %.2e" % (np.abs(host(y) - ys).max(), bound), flush=True)
        assert np.abs(host(y) - ys).max() <= bound
        for name, a, b in zip(("dtheta", "dx", "dy0"), ctx.grad(th, xd, y0d, dev(ys, 0), dev(g, 0)), want):
            assert np.abs(host(a).reshape(-1) - b.reshape(-1)).max() <= 1e-4 * max(1.0, np.abs(b).max()), (name, np.abs(host(a).reshape(-1) - b.reshape(-1)).max())
    finally:
        ctx.close()


# the same at the chunk length the dispatch takes by itself: with 64 sequences of 100,000 positions nothing but a limit keeps the chunks short (a step
# multiplies by two: 2^127 is the largest power)
@pytest.mark.parametrize("kind,n", [("gru", 16), ("gru", 8)])
def test_expanding_jacobians_at_the_default_chunk_length(kind, n):
    B, T = 64, 100000
    theta = np.concatenate([np.zeros(3 * n + 2 * n * n), 6.0 * np.eye(n).ravel(), np.zeros(4 * n)])
    ctx = deer.DeerContext(deer.make_config(deer.DEER_CELL_GRU, deer.DEER_F32, B, T, n, d=1), device=DEV)
    try:
        y, it, _, conv, st = ctx.eval(dev(theta, 0), torch.zeros(B, T, 1, device=DEV), torch.zeros(B, n, device=DEV), tol=1e-6, max_iter=5)
        assert st == deer.DEER_OK and conv and it == 1 and not y.any()
    finally:
        ctx.close()


# the maps of the chunks lie where the recurrence alone publishes its words: calls of one context in any order, and a gradient that a knob keeps on the scans
@pytest.mark.parametrize("n,d", [(8, 4), (16, 6), (32, 8), (64, 5)])
def test_recurrence_alone_between_steps_by_chunks(n, d, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", "8")
    if n > 8:
        monkeypatch.setenv("DEER_GRAD_FUSED", "0")
    B, T = 3, 2500
    w = inputs.gru_workload("between_n%d" % n, 3300 + n, B=B, T=T, n=n, d=d)
    rng = np.random.default_rng(n)
    A, b, v = dev(rng.standard_normal((B, T, n, n)) * 0.45 / np.sqrt(n), 0), dev(rng.standard_normal((B, T, n)), 0), dev(rng.standard_normal((B, n)), 0)
    g = dev(rng.standard_normal((B, T, n)) / T, 0)
    th, x, y0 = dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0)
    ctx = deer.context_for(w, device=DEV)
    try:
        first, back = ctx.linrec_solve(A, b, v), ctx.linrec_solve(A, b, reverse=True)
        y = ctx.eval(th, x, y0, tol=w.tol, max_iter=w.max_iter)[0]
        grads = ctx.grad(th, x, y0, y, g)
        for _ in range(2):
            assert torch.equal(ctx.linrec_solve(A, b, v), first)
            assert torch.equal(ctx.eval(th, x, y0, tol=w.tol, max_iter=w.max_iter)[0], y)
            assert torch.equal(ctx.linrec_solve(A, b, reverse=True), back)
            assert all(torch.equal(p, q) for p, q in zip(ctx.grad(th, x, y0, y, g), grads))
    finally:
        ctx.close()


# the routes that the dispatch takes by itself: plain n = 8 by chunks (from 380,000 positions), on the scan (up to 512 tiles there), in one launch, each with
# the gradient by chunks; heads on the scan with their gradient by chunks (one tile a compute unit) and by chunks; the LEM of 8 units with the gradient alone by chunks
@pytest.mark.parametrize("kind,n,d,B,T,H,K", [("gru", 8, 4, 40, 9501, 0, 0), ("gru", 7, 3, 21, 18103, 0, 0), ("gru", 8, 4, 16, 2049, 0, 0), ("heads", 8, 4, 2, 4001, 8, 1),
                                              ("heads", 8, 8, 9, 903, 11, 3), ("lem", 8, 4, 40, 211, 0, 0), ("lem", 8, 4, 1, 2501, 0, 0)])
def test_routes_of_the_dispatch(kind, n, d, B, T, H, K):
    if kind == "heads":
        w = inputs.mh_gru_workload("route_mh", 3400 + T, B=B, T=T, n=n, d=d, H=H, K=K)
        solve = lambda m: oracle.mh_deer_eval(n, d, H, K, w.theta, w.x, w.y0, tol=w.tol, max_iter=m, nthreads=8)
        seq, grad = lambda: oracle.mh_seq_eval(n, d, H, K, w.theta, w.x, w.y0, nthreads=8), lambda ys, g: oracle.mh_gru_grad(n, d, H, K, w.theta, w.x, w.y0, ys, g)
    else:
        w = (inputs.gru_workload("route", 3400 + T, B=B, T=T, n=n, d=d) if kind == "gru" else inputs.lem_workload("route", 3400 + T, B=B, T=T, units=n, d=d))
        c = oracle_cell(w) if kind == "gru" else oracle.make_cell(oracle.CELL_LEM, 2 * n, d, dt=w.t1)
        solve = lambda m: oracle.deer_eval(c, w.theta, w.x, w.y0, tol=w.tol, max_iter=m, nthreads=8)
        seq = lambda: oracle.seq_eval(c, w.theta, w.x, w.y0, nthreads=8)
        grad = lambda ys, g: (oracle.gru_grad(w.n, w.d, w.theta, w.x, w.y0, ys, g) if kind == "gru" else oracle.rnn_grad(c, w.theta, w.x, w.y0, ys, g))
    ctx = deer.context_for(w, device=DEV)
    try:
        ctx.set_profiling(True)
        _against_oracle(ctx, w, solve, seq, grad)
        p = ctx.profile()
        # which kernels ran: a launch per iteration by chunks or on the multi-head scan, a whole solve in one launch, or Jacobian kernel and scan;
        # where the gradient goes by chunks there is no launch of a vector-Jacobian product
        one_launch = kind == "gru" and T == 2049
        assert p["vjp_launches"] == 0 and (p["newton_launches"] > 0) == one_launch
        assert (p["scan_launches"] > 0) == (kind == "lem" and T == 211) and (p["fused_launches"] > 1) == (not one_launch and not (kind == "lem" and T == 211))
    finally:
        ctx.close()


# Solves whose iterates pass through values of 1e16 to 1e37 before they converge (by the oracle): the next iterate comes from one that is larger by
# 1e15 and more, which leaves nothing of a correction.  The count of such iterations depends on every rounding, the solution does not.
@pytest.mark.parametrize("kind,n,scale,seed", [("lem", 9, 1.0, 1887), ("lstm", 8, 1.5, 5012), ("lstm", 16, 2.5, 5005), ("gru", 8, 1.5, 5012), ("gru", 8, 2.5, 5009), ("gru", 16, 2.5, 5012),
                                               ("heads", 8, 1.5, 5012), ("heads", 8, 2.5, 5009)])
@pytest.mark.parametrize("L", ["4", "32"])
def test_iterates_far_from_the_solution(kind, n, scale, seed, L, monkeypatch):
    monkeypatch.setenv("DEER_CHUNK_L", L)
    if kind == "heads":
        w = inputs.mh_gru_workload("far", seed, B=6, T=1252, n=n, d=2, H=3, K=2)
    elif kind == "lem":
        w = inputs.lem_workload("far", seed, B=3, T=1543, units=n, d=1)
        w.y0 = (np.random.default_rng(7).standard_normal((3, 2 * n)) * 0.5).astype(np.float32)
    else:
        w = (inputs.gru_workload("far", seed, B=6, T=1252, n=n, d=2) if kind == "gru" else inputs.lstm_workload("far", seed, B=6, T=1252, units=n, d=2))
    w.theta = (w.theta * np.float32(scale)).astype(np.float32)
    if kind == "heads":
        _, ito, erro, hist = oracle.mh_deer_eval(n, 2, 3, 2, w.theta, w.x, w.y0, tol=1e-4, max_iter=100, nthreads=8)
        ys = oracle.mh_seq_eval(n, 2, 3, 2, w.theta, w.x, w.y0, nthreads=8)
    else:
        c = oracle.make_cell({"gru": oracle.CELL_GRU, "lstm": oracle.CELL_LSTM, "lem": oracle.CELL_LEM}[kind], n if kind == "gru" else 2 * n, w.d, **({"dt": w.t1} if kind == "lem" else {}))
        _, ito, erro, hist = oracle.deer_eval(c, w.theta, w.x, w.y0, tol=1e-4, max_iter=100, nthreads=8)
        ys = oracle.seq_eval(c, w.theta, w.x, w.y0, nthreads=8)
    assert erro <= 1e-4 and np.nanmax(hist) > 1e10
    ctx = deer.context_for(w, device=DEV)
    try:
        y, it, _, conv, st = ctx.eval(dev(w.theta, 0), dev(w.x, 0), dev(w.y0, 0), tol=1e-4, max_iter=200)
        print(kind, n, "%d iterations (oracle %d, largest step %.1e)" % (it, ito, np.nanmax(hist)), np.abs(host(y) - ys).max(), flush=True)
        assert st == deer.DEER_OK and conv
        assert np.abs(host(y) - ys).max() <= 1e-4   # (weights off by one in 2^24 change these solutions by 2e-6 at most)
    finally:
        ctx.close()
