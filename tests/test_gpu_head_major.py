"""GPU parity of the multi-head steps that run on transposed copies of the input and the iterates (large layers of three stride levels and more)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_12252_amd import deer, inputs
from helpers import DEV, dev, host

pytestmark = pytest.mark.gpu


# rows of whole 16-byte pieces and of three scalars, times that are no multiple of a tile, an input that is only scalar-aligned, more sequences than a grid's
# second dimension takes; the last one is large enough for copies from a guess too
@pytest.mark.parametrize("B,T,H,K,d,shift", [(37, 1001, 32, 3, 4, 0), (49, 1001, 32, 4, 3, 0), (37, 1001, 32, 8, 4, 1), (70001, 8, 4, 3, 4, 0), (61, 3901, 32, 3, 4, 1)])
def test_large_layers(B, T, H, K, d, shift):
    n = 8
    w = inputs.mh_gru_workload("head_major", 51 + d, B=B, T=T, n=n, d=d, H=H, K=K)
    w.y0 = (np.random.default_rng(d).standard_normal((B, H, n)) * 0.5).astype(np.float32)
    want = oracle.mh_seq_eval(n, d, H, K, w.theta, w.x, w.y0, nthreads=8)
    x = torch.empty(w.x.size + shift, device=DEV)[shift:].view(B, T, H, d)
    x.copy_(dev(w.x, 0))
    ctx = deer.context_for(w, device=DEV)
    try:
        th, y0 = dev(w.theta, 0), dev(w.y0, 0)
        y, it, _, conv, st = ctx.eval(th, x, y0, tol=w.tol, max_iter=w.max_iter)
        assert st == deer.DEER_OK and conv and np.abs(host(y) - want).max() <= 1e-4
        # from a guess (the solution: one more step of about its rounding), and cut short: the last iterate comes back in the caller's layout
        z, again, err, conv, st = ctx.eval(th, x, y0, y_guess=y, tol=w.tol, max_iter=w.max_iter)
        assert st == deer.DEER_OK and conv and again == 1 and err <= 1e-5 and np.abs(host(z) - want).max() <= 1e-4
        if y.numel() > 5e7:
            return   # (the oracle of one step stores its Jacobians)
        first = ctx.eval(th, x, y0, tol=w.tol, max_iter=1)[0]
        few = oracle.mh_deer_eval(n, d, H, K, w.theta, w.x, w.y0, tol=w.tol, max_iter=1, nthreads=8)[0]
        assert np.abs(host(first) - few).max() <= 1e-4
    finally:
        ctx.close()
