"""The last 3x3 decoder layer's own kernel (up to 32 channels, a multiple of 8)
against the general convolution: the same network padded to 40 channels that
are zero has no such kernel and gives the same map but for rounding."""
import numpy as np
import pytest
import torch

from tests.gpu_util import cuda, flat_params, normwise, vae_params

pytestmark = pytest.mark.gpu


def _padded(params, c1, c2, z):
    """The same network with z zero channels after E1's, G1's and G0's."""
    p = [(w.copy(), b.copy()) for w, b in params]

    def outs(i):
        w, b = p[i]
        p[i] = (np.concatenate([w, np.zeros((z,) + w.shape[1:], w.dtype)]), np.concatenate([b, np.zeros(z, b.dtype)]))

    def ins(i, at):
        w, b = p[i]
        p[i] = (np.insert(w, [at] * z, 0.0, axis=1), b)

    for i in (0, 6, 7):
        outs(i)
    ins(1, c1)
    ins(6, c2 + c1)
    ins(7, c1)
    ins(8, c1)
    return p


def _forward(c1, dtype, params, disp, img, H, W, f):
    import paper_2305_11566_amd as sv
    ref = sv.Refiner(c1, 32, 48, 32, f, dtype)
    ref.pack(cuda(flat_params(params)))
    out, _ = ref.forward(cuda(disp), cuda(img), H, W)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# A 16-bit value that falls on another side of a rounding moves by one unit, a
# part of 2^-7 (bf16) or 2^-10 (f16) of itself; both layers that read maps in
# 16 bits after the first difference may add one.  INT8 sums are whole numbers:
# only the FP32 projection's order is left.
TOL = {"bf16": 2 * 2.0 ** -7, "f16": 2 * 2.0 ** -10, "i8": 1e-5}


@pytest.mark.parametrize("H,W,f,B", [
    (8, 8, 8, 2),       # a map of one pixel
    (45, 61, 4, 3),     # 12x16: one tile column, an odd level below
    (66, 130, 2, 2),    # 33x65: one past the tiles' edges
    (70, 62, 2, 40),    # 35x31, images enough for several tiles a workgroup
])
@pytest.mark.parametrize("c1", [8, 16, 24, 32])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "i8"])
def test_g0_kernel_against_general(dtype, c1, H, W, f, B):
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(c1 + H)
    h, w = -(-H // f), -(-W // f)
    disp = rng.integers(0, 48, (B, h, w)).astype(np.uint8)
    img = rng.integers(0, 256, (B, h, w)).astype(np.uint8)
    params = vae_params((c1, 32, 48), 32, 900 + c1)
    names = [sv.sv_conv_cfg_name(c) for c in range(sv.sv_num_layer_cfgs())]
    want = _forward(40, dtype, _padded(params, c1, 32, 40 - c1), disp, img, H, W, f)
    first = None
    try:
        for tile in (None, "th4_tn16", "th8_tn32", "th16_tn32"):
            sv.sv_set_layer_cfg(7, -1 if tile is None else names.index(tile))
            got = _forward(c1, dtype, params, disp, img, H, W, f)
            first = got if first is None else first
            assert np.array_equal(got, first), f"{tile}: not the default tile's bits"
    finally:
        sv.sv_set_layer_cfg(7, -1)
    assert normwise(first, want) <= TOL[dtype]
