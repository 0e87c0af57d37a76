"""The upsampling layer's input gradient: the feature layers' weight gradients
hang on it, so a backward of a network whose other paths into them are closed (the
encoder's and decoder's weights zero) is held against 64 bits."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu

# FP32 sums of 25 products and of h w pixels beside each other; 16 bits: the
# weight gradients' operands are rounded to the type
TOL = {"f32": 1e-5, "bf16": 2.0 ** -7, "f16": 2.0 ** -10}


@pytest.mark.parametrize("h,w,f,B", [(1, 1, 4, 1), (5, 13, 2, 1), (33, 47, 3, 3)])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_upsampling_input_gradient(dtype, h, w, f, B):
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(h * w + f)
    es = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    disp = torch.from_numpy(rng.integers(0, 60, (B, h, w)).astype(np.uint8))
    img = torch.from_numpy(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    net = sv.TableVAE(f, dtype)
    params = torch.zeros(net.nparams)
    # FE_1, FE_2: positive weights keep every output positive (no sign flips)
    params[:1664] = torch.from_numpy(rng.uniform(0.05, 0.2, 1664).astype(np.float32)).to(es).float()
    params[-2026:] = torch.from_numpy(rng.normal(0, 0.1, 2026).astype(np.float32))
    net.pack(params.cuda())
    H, W = h * f, w * f
    dout = torch.from_numpy(rng.normal(0, 1, (B, H, W)).astype(np.float32))
    d, i = cuda(disp.numpy()), cuda(img.numpy())
    net.forward(d, i, H, W)
    grad = net.backward(d, i, H, W, dout.cuda()).double().cpu()
    torch.cuda.synchronize()
    # 64 bits: out = 256 convT(FE, w) + ..., so dFE = 256 conv(dout, w), stride f
    wy = params[-2026:-1].double().reshape(81, 1, 5, 5)[17:]  # FE's rows of [D | X_0 | FE]
    dfe = 256 * F.conv2d(F.pad(dout.double()[:, None], (2, 2 + f, 2, 2 + f)), wy, stride=f)[:, :, :h, :w]
    for c, x in enumerate((disp.double() * f / 256, img.double() / 256)):
        dy = dfe[:, 32 * c:32 * c + 32]
        cols = F.unfold(x[:, None], 5, padding=2)                     # [B, 25, h w]
        want = torch.einsum("bok,btk->ot", dy.flatten(2), cols).flatten()
        size = torch.einsum("bok,btk->ot", dy.flatten(2).abs(), cols).flatten()
        got = grad[c * 832:c * 832 + 800]
        assert float(((got - want).abs() / size.clamp_min(1e-30)).max()) <= TOL[dtype]
