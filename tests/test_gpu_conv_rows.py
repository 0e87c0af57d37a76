"""The row kernel (5x5 and 3x3 layers that read one map in place, 3x3 ones of a
resized map) against the general convolution, taken at another tile shape or a
smaller batch: the same bits."""
import numpy as np
import pytest
import torch

from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,B", [
    (2, 3, 3),        # too few workgroups on every level: the general kernel
    (33, 66, 20),     # one row a wave on some levels, remainders past every tile
    (127, 129, 9),    # two rows a wave, ragged
    (130, 250, 31),   # four rows a wave, ragged
])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_rows_equal_general_bitwise(dtype, h, w, B):
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(h + w)
    disp = cuda(rng.integers(0, 48, (B, h, w)).astype(np.uint8))
    img = cuda(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    net = sv.TableVAE(1, dtype)
    net.pack(cuda(rng.normal(0, 0.05, net.nparams).astype(np.float32)))
    names = [sv.sv_conv_cfg_name(c) for c in range(sv.sv_num_layer_cfgs())]
    outs = []
    try:
        for tile in ("th4_tn16", "th8_tn16_k2", "th4_tn32"):
            for layer in range(sv.sv_tvae_num_layers()):
                sv.sv_tvae_set_layer_cfg(layer, names.index(tile))
            out, _ = net.forward(disp, img, h, w)
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
    finally:
        for layer in range(sv.sv_tvae_num_layers()):
            sv.sv_tvae_set_layer_cfg(layer, -1)
    assert np.array_equal(outs[0], outs[1])
    assert np.array_equal(outs[2], outs[1])


@pytest.mark.parametrize("f,c,H,W", [
    (2, (16, 32, 64), 66, 130),   # 33x65: one past the tiles' edges on every level
    (1, (8, 24, 40), 61, 47),     # partial chunks and channel blocks
])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_3x3_rows_equal_general(dtype, f, c, H, W):
    """24 copies of an image in a training pass take the kernel at four, two and
    (FP32) one row a wave, one image alone the general one: the same map, and 24
    times the gradient but for the order of its FP32 sums over pixels."""
    import paper_2305_11566_amd as sv
    B = 24
    rng = np.random.default_rng(H)
    h, w = -(-H // f), -(-W // f)
    disp = rng.integers(0, 48, (1, h, w)).astype(np.uint8)
    img = rng.integers(0, 256, (1, h, w)).astype(np.uint8)
    ref = sv.Refiner(*c, 32, f, dtype)
    ref.pack(cuda(rng.normal(0, 0.1, ref.nparams).astype(np.float32)))
    eps1 = rng.normal(0, 1, ref.latent_shape(1, H, W)).astype(np.float32)
    dout1 = rng.normal(0, 1, (1, H, W)).astype(np.float32)
    names = [sv.sv_conv_cfg_name(k) for k in range(sv.sv_num_layer_cfgs())]
    res = []
    try:
        for layer in range(1, 8):
            sv.sv_set_layer_cfg(layer, names.index("th4_tn16"))
        for n in (1, B):
            d, i, e, g = (cuda(np.repeat(a, n, 0)) for a in (disp, img, eps1, dout1))
            saved = ref.saved_buffer(n, H, W)
            out, _ = ref.forward(d, i, H, W, eps=e, saved=saved)
            grad = ref.backward(saved, n, H, W, e, g, 0.0)
            torch.cuda.synchronize()
            res.append((out.cpu().numpy(), grad.double().cpu().numpy() / n))
    finally:
        for layer in range(1, 8):
            sv.sv_set_layer_cfg(layer, -1)
    (o1, g1), (ob, gb) = res
    assert all(np.array_equal(o1[0], o) for o in ob)
    assert np.abs(g1 - gb).max() <= 1e-5 * np.abs(g1).max()


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_3x3_rows_at_the_default_tile_only(dtype):
    """The row kernel stands for the default tiles, a set tile is the general kernel's:
    both give the map and the gradient of a training pass of 24 images."""
    import paper_2305_11566_amd as sv
    B, H, W, f, c = 24, 66, 130, 2, (16, 32, 64)
    rng = np.random.default_rng(5)
    h, w = -(-H // f), -(-W // f)
    disp = cuda(rng.integers(0, 48, (B, h, w)).astype(np.uint8))
    img = cuda(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    ref = sv.Refiner(*c, 32, f, dtype)
    ref.pack(cuda(rng.normal(0, 0.1, ref.nparams).astype(np.float32)))
    eps = cuda(rng.normal(0, 1, ref.latent_shape(B, H, W)).astype(np.float32))
    dout = cuda(rng.normal(0, 1, (B, H, W)).astype(np.float32))
    names = [sv.sv_conv_cfg_name(k) for k in range(sv.sv_num_layer_cfgs())]
    res = []
    try:
        for tile in (None, "th8_tn16_k2", "th4_tn16"):
            for layer in range(1, 8):
                sv.sv_set_layer_cfg(layer, names.index(tile) if tile else -1)
            saved = ref.saved_buffer(B, H, W)
            out, _ = ref.forward(disp, img, H, W, eps=eps, saved=saved)
            grad = ref.backward(saved, B, H, W, eps, dout, 0.0)
            torch.cuda.synchronize()
            res.append((out.cpu().numpy(), grad.cpu().numpy()))
    finally:
        for layer in range(1, 8):
            sv.sv_set_layer_cfg(layer, -1)
    for out, grad in res[1:]:
        assert np.array_equal(out, res[0][0]) and np.array_equal(grad, res[0][1])
