"""The adjoints of the final layer and of the resizes at every reduction factor
and at the edges of their tiles (32 coarse columns, 8 / 4 / 2 coarse rows by the
factor), against the oracle's FP64 gradient: FP32 1e-4 normwise per layer, as
in the backward's other parity tests."""
import numpy as np
import pytest

from oracle import vae
from synth import gen_eps
from tests.gpu_util import normwise, vae_params
from tests.test_gpu_train import _gpu_grad, _layer_slices, _oracle_grad, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f,H,W", [
    (1, 9, 33), (2, 33, 65), (3, 26, 101), (4, 17, 129), (5, 21, 166), (6, 37, 67), (7, 29, 230), (8, 57, 263),
    (8, 3, 5), (3, 1, 1),
])
def test_every_factor(f, H, W):
    C, L, B = (8, 16, 8), 8, 2
    disp, img, gt = _problem(H, W, f, C, L, B, seed=700 + f)
    params = vae_params(C, L, seed=30 + f)
    eps = gen_eps((B, -(-H // (8 * f)), -(-W // (8 * f)), L), seed=f)
    g_or, dout, _ = _oracle_grad(params, disp, img, f, H, W, eps, gt, 0.25)
    g_gpu, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, eps, dout, 0.25)
    for name, sl in zip(vae.LAYERS, _layer_slices(C, L)):
        e = normwise(g_gpu[sl], g_or[sl])
        assert e <= 1e-4, f"{name}: normwise {e:.2e}"


def test_a_gradient_that_is_not_finite_stays_where_it_is_read():
    """One infinite entry of dout reaches the parameters' gradient as infinity
    or NaN, and an image without it keeps a finite one."""
    f, H, W, C, L = 2, 40, 70, (8, 16, 8), 8
    disp, img, gt = _problem(H, W, f, C, L, 1, seed=5)
    params = vae_params(C, L, seed=6)
    dout = np.random.default_rng(1).standard_normal((1, H, W))
    a, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, None, dout, 0.0)
    assert np.isfinite(a).all()
    dout[0, 11, 13] = np.inf
    b, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, None, dout, 0.0)
    assert not np.isfinite(b).all()


@pytest.mark.parametrize("f,H,W", [(2, 40, 70), (4, 37, 129), (7, 30, 45)])
def test_an_infinity_at_the_edge_stays_out_of_the_taps_that_do_not_read_it(f, H, W):
    """dout's last column is read by the final layer's taps of the columns before and at
    it (of three), its last row likewise: the others' weight gradients stay finite."""
    C, L = (8, 16, 8), 8
    disp, img, gt = _problem(H, W, f, C, L, 1, seed=8)
    params = vae_params(C, L, seed=9)
    for y, x, clean in ((H // 2, W - 1, np.s_[:, :, 2]), (H - 1, W // 2, np.s_[:, 2, :]),
                        (H // 2, 0, np.s_[:, :, 0]), (0, W // 2, np.s_[:, 0, :])):
        dout = np.random.default_rng(2).standard_normal((1, H, W))
        dout[0, y, x] = np.inf
        g, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, None, dout, 0.0)
        dw = g[_layer_slices(C, L)[-1]][:-1].reshape(C[0] + 2, 3, 3)
        keep = np.zeros((C[0] + 2, 3, 3), bool)
        keep[clean] = True
        assert np.isfinite(dw[keep]).all(), (y, x)
        assert not np.isfinite(dw[~keep]).any(), (y, x)
