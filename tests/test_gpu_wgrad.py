"""The weight-gradient kernels at the edges of their tiles (8 or 4 rows x 16
columns of output pixels, 16 or 32 channels and rows a workgroup, more tiles
than workgroups) against the oracle's FP64 gradient.  The bars are those of
the backward's other parity tests: FP32 1e-4 normwise per layer."""
import numpy as np
import pytest
import torch

from oracle import vae
from synth import gen_eps
from tests.gpu_util import cuda, normwise, vae_params
from tests.test_gpu_train import _gpu_grad, _layer_slices, _oracle_grad, _problem
from tests.test_gpu_tvae import test_f32_gradients_match_oracle as _table_gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,f,C,L,B", [
    (17, 33, 1, (16, 32, 40), 24, 1),    # one pixel past the tiles, a third chunk of rows
    (34, 62, 2, (32, 48, 16), 40, 3),    # one row past two tiles, 31 columns, three chunks of channels
    (9, 200, 1, (8, 24, 8), 8, 2),       # single-row coarse levels
    (770, 1026, 2, (8, 8, 8), 8, 1),     # more tiles than workgroups, ragged in both directions
])
def test_refiner_f32(H, W, f, C, L, B):
    disp, img, gt = _problem(H, W, f, C, L, B, seed=600 + H)
    params = vae_params(C, L, seed=H + 3 * W)
    h3, w3 = -(-H // (8 * f)), -(-W // (8 * f))
    eps = gen_eps((B, h3, w3, L), seed=H)
    g_or, dout, _ = _oracle_grad(params, disp, img, f, H, W, eps, gt, 0.25)
    g_gpu, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, eps, dout, 0.25)
    for name, sl in zip(vae.LAYERS, _layer_slices(C, L)):
        e = normwise(g_gpu[sl], g_or[sl])
        assert e <= 1e-4, f"{name}: normwise {e:.2e}"


@pytest.mark.parametrize("f,H,W,B", [
    (1, 17, 35, 1),      # one past the tiles at every level
    (2, 66, 30, 3),
])
def test_table_f32(f, H, W, B):
    _table_gradients(f, H, W, B, True)


def test_table_f32_more_tiles_than_workgroups():
    """64 copies of an image in one batch (25 tiles each at level 1, more than
    there are workgroups) give 64 times its gradient."""
    import paper_2305_11566_amd as sv
    f, H, W, n = 2, 66, 130, 64
    r = np.random.default_rng(17)
    d = r.integers(0, 40, (1, 33, 65)).astype(np.uint8)
    im = r.integers(0, 256, (1, 33, 65)).astype(np.uint8)
    dout = r.standard_normal((1, H, W)).astype(np.float32)
    net = sv.TableVAE(f, "f32")
    net.pack(torch.randn(net.nparams, generator=torch.Generator().manual_seed(3)).mul_(0.05).cuda())
    g = []
    for k in (1, n):
        dd, ii, do = (cuda(np.repeat(a, k, axis=0)) for a in (d, im, dout))
        net.forward(dd, ii, H, W)
        g.append(net.backward(dd, ii, H, W, do).cpu().numpy().astype(np.float64))
    assert normwise(g[1], n * g[0]) <= 1e-4


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_refiner_16bit_ragged(dtype):
    """Against the FP32 gradient of the same weights: cosine per layer as in the
    backward's own 16-bit test, at ragged sizes."""
    H, W, f, C, L, B = 98, 130, 2, (16, 32, 40), 24, 3
    disp, img, gt = _problem(H, W, f, C, L, B, seed=81)
    params = vae_params(C, L, seed=9)
    dout = np.random.default_rng(5).standard_normal((B, H, W)) / (B * H * W)
    eps = gen_eps((B, -(-H // 16), -(-W // 16), L), seed=12)
    g32, _ = _gpu_grad(C, L, f, "f32", params, disp, img, H, W, eps, dout, 0.25)
    g16, _ = _gpu_grad(C, L, f, dtype, params, disp, img, H, W, eps, dout, 0.25)
    for name, sl in zip(vae.LAYERS, _layer_slices(C, L)):
        a, b = g32[sl], g16[sl]
        cos = float(a @ b / max(np.linalg.norm(a) * np.linalg.norm(b), 1e-30))
        assert cos >= 0.99, f"{name}: cosine {cos:.5f}"
