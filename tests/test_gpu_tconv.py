"""The transposed convolutions' own kernel against the general convolution over
the zero-inserted map: the sums have the same order, so the results are the same
bits.  (Its other use, the stride-2 layers' input gradients, is held against the
oracle by the gradient tests of both networks.)"""
import numpy as np
import pytest
import torch

from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,B", [
    (1, 1, 1),        # one pixel on every level
    (6, 5, 2),        # 3x3 and 2x2 below: odd and even outputs
    (67, 66, 1),      # 34x33: one past a tile; one row a workgroup
    (35, 129, 5),     # two rows a workgroup on level 1
    (64, 96, 24),     # four rows a workgroup on level 1, two on level 2
    (131, 250, 14),   # four rows a workgroup on both
])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_deconvolutions_equal_zero_inserted_bitwise(dtype, h, w, B):
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(h + w)
    disp = cuda(rng.integers(0, 48, (B, h, w)).astype(np.uint8))
    img = cuda(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    net = sv.TableVAE(1, dtype)
    net.pack(cuda(rng.normal(0, 0.05, net.nparams).astype(np.float32)))
    names = [sv.sv_conv_cfg_name(c) for c in range(sv.sv_num_layer_cfgs())]
    outs = []
    try:
        for layer in range(sv.sv_tvae_num_layers()):
            sv.sv_tvae_set_layer_cfg(layer, names.index("th4_tn16"))  # no split reductions
        for form in (0, -1):
            sv.sv_tvae_set_deconv_form(form)
            out, _ = net.forward(disp, img, h, w)
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
    finally:
        sv.sv_tvae_set_deconv_form(-1)
        for layer in range(sv.sv_tvae_num_layers()):
            sv.sv_tvae_set_layer_cfg(layer, -1)
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_small_16_bit_grids_keep_their_split(dtype):
    """Where the layers' configurations split the reduction, 16-bit passes take the
    zero-inserted form by default too."""
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(11)
    h, w = 40, 52
    disp = cuda(rng.integers(0, 48, (1, h, w)).astype(np.uint8))
    img = cuda(rng.integers(0, 256, (1, h, w)).astype(np.uint8))
    net = sv.TableVAE(1, dtype)
    net.pack(cuda(rng.normal(0, 0.05, net.nparams).astype(np.float32)))
    outs = []
    try:
        for form in (0, -1):
            sv.sv_tvae_set_deconv_form(form)
            out, _ = net.forward(disp, img, h, w)
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
    finally:
        sv.sv_tvae_set_deconv_form(-1)
    assert np.array_equal(outs[0], outs[1])


def test_maps_past_32_bit_offsets_take_the_general_kernel():
    """From 2^31 elements an image's map is past the kernel's offsets (level 2 of one
    13400x13400 image at factor 1): the pass runs, as the zero-inserted form does."""
    import paper_2305_11566_amd as sv
    H = W = 13400
    assert 48 * (H // 2) * (W // 2) >= 2 ** 31
    gen = torch.Generator(device="cuda").manual_seed(7)
    disp = torch.randint(0, 48, (1, H, W), dtype=torch.uint8, device="cuda", generator=gen)
    img = torch.randint(0, 256, (1, H, W), dtype=torch.uint8, device="cuda", generator=gen)
    net = sv.TableVAE(1, "bf16")
    net.pack(cuda(np.random.default_rng(3).normal(0, 0.05, net.nparams).astype(np.float32)))
    out, _ = net.forward(disp, img, H, W)
    try:
        sv.sv_tvae_set_deconv_form(0)
        want, _ = net.forward(disp, img, H, W)
    finally:
        sv.sv_tvae_set_deconv_form(-1)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
