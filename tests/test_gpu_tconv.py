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
