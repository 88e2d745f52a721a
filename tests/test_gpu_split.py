"""GPU parity of the kernels that run fp32 products on the fp16 matrix cores (factors split in two), where the split or its scaling
can go wrong: remainders, weights far from one, activations far from one, zero layers."""
import numpy as np
import pytest

from paper_2309_12252_amd import deer, inputs
from helpers import TOL_ABS
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


CASES = [(width, nhid, act, plain) for width in (32, 64) for nhid, act in
         ((1, inputs.ACT_SOFTPLUS), (2, inputs.ACT_SOFTPLUS), (3, inputs.ACT_TANH), (4, inputs.ACT_SOFTPLUS), (5, inputs.ACT_TANH))]
CASES += [(64, 4, inputs.ACT_TANH, far_scales), (32, 3, inputs.ACT_TANH, far_scales), (64, 5, inputs.ACT_SOFTPLUS, large_activations),
          (32, 2, inputs.ACT_SOFTPLUS, large_activations), (64, 3, inputs.ACT_TANH, zero_layer), (32, 5, inputs.ACT_SOFTPLUS, zero_layer)]


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
