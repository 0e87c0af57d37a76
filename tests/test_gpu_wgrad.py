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


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n", [12, 64])
def test_table_16bit_large_batches(dtype, n):
    """12 and 64 copies of an image take the 16-bit input gradients to the row kernel
    and the transposed convolution at two and four rows, one image alone to the general
    kernel and to one row: the same gradient maps, so n times the gradient but for the
    order of its FP32 sums (the FP32 bar of the backward's parity tests, per layer)."""
    import paper_2305_11566_amd as sv
    f, H, W = 2, 132, 260
    r = np.random.default_rng(19)
    d = r.integers(0, 40, (1, H // f, W // f)).astype(np.uint8)
    im = r.integers(0, 256, (1, H // f, W // f)).astype(np.uint8)
    dout = r.standard_normal((1, H, W)).astype(np.float32)
    eps = r.standard_normal((1, 17, 33)).astype(np.float32)
    net = sv.TableVAE(f, dtype)
    net.pack(torch.randn(net.nparams, generator=torch.Generator().manual_seed(4)).mul_(0.05).cuda())
    names = [sv.sv_conv_cfg_name(c) for c in range(sv.sv_num_layer_cfgs())]
    res = []
    try:
        for layer in range(sv.sv_tvae_num_layers()):  # no split reductions: the same maps at both sizes
            sv.sv_tvae_set_layer_cfg(layer, names.index("th4_tn16"))
        for k in (1, n):
            dd, ii, do, ee = (cuda(np.repeat(a, k, axis=0)) for a in (d, im, dout, eps))
            out, _ = net.forward(dd, ii, H, W, eps=ee)
            g = net.backward(dd, ii, H, W, do, eps=ee)
            res.append((out.cpu().numpy(), g.cpu().numpy().astype(np.float64)))
    finally:
        for layer in range(sv.sv_tvae_num_layers()):
            sv.sv_tvae_set_layer_cfg(layer, -1)
    assert (res[1][0] == res[0][0]).all()
    at = 0
    for o, c, k in [(32, 1, 5), (32, 1, 5), (16, 64, 5), (8, 16, 5), (32, 24, 5), (16, 32, 5), (2, 48, 1), (32, 1, 1),
                    (16, 80, 5), (16, 96, 5), (8, 40, 5), (16, 48, 5), (1, 81, 5)]:
        sl = slice(at, at + o * c * k * k + o)
        assert normwise(res[1][1][sl], n * res[0][1][sl]) <= 1e-4, (at, o, c, k)
        at = sl.stop
