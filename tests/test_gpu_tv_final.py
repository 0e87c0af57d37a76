"""The upsampling layer's kernel (tap projections and gather in one) against the
transposed convolution in 64 bits of the level-1 map the same pass stored: only
FP32 rounding is left between the two, also for maps in 16 bits."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-5  # the FP32 bar of this network's other tests
ES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


@pytest.mark.parametrize("H,W,f,B", [
    (1, 1, 8, 1),        # one level-1 pixel
    (9, 17, 1, 2),       # one past the tile, halos on both sides
    (33, 66, 2, 3),      # 17x33, likewise
    (25, 50, 3, 1),      # a factor without a kernel of its own
    (96, 190, 4, 1),     # 24x48: whole tiles
    (41, 133, 4, 90),    # tiles enough for several a workgroup
])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_upsampling_against_64_bits(dtype, H, W, f, B):
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(H * W + f)
    h, w = -(-H // f), -(-W // f)
    disp = torch.from_numpy(rng.integers(0, 60, (B, h, w)).astype(np.uint8))
    img = torch.from_numpy(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    net = sv.TableVAE(f, dtype)
    params = torch.from_numpy(rng.normal(0, 0.1, net.nparams).astype(np.float32))
    net.pack(params.cuda())
    out, _ = net.forward(cuda(disp.numpy()), cuda(img.numpy()), H, W)
    torch.cuda.synchronize()
    es = ES[dtype]
    # the level-1 map [D 16 | FE 64] opens the workspace
    l1 = net.workspace(B, H, W)[:B * h * w * 80 * es.itemsize].view(es).reshape(B, h, w, 80)
    l1 = l1.double().cpu().permute(0, 3, 1, 2)
    x0 = disp.double()[:, None] * f / 256
    wy = params[-2026:-1].double().reshape(81, 1, 5, 5)  # over [D | X_0 | FE]
    cat = F.pad(torch.cat([l1[:, :16], x0, l1[:, 16:]], 1), (0, 2, 0, 2))
    want = 256 * (F.conv_transpose2d(cat, wy, stride=f, padding=2)[:, 0, :H, :W] + params[-1].double())
    err = float((out.double().cpu() - want).abs().max() / want.abs().max())
    assert err <= TOL_F32, f"normwise {err:.3e}"
