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


# FP32: a chain of 25 roundings and the bias, half a unit each; 16 bits: the
# stored value's rounding on top
FE_TOL = {"f32": 26 * 2.0 ** -24, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}


@pytest.mark.parametrize("h,w,f,B", [(1, 1, 4, 1), (5, 17, 2, 2), (45, 33, 3, 70), (16, 16, 1, 512)])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_feature_extraction_against_64_bits(dtype, h, w, f, B):
    """Four rows a workgroup and (from 512 workgroups) sixteen, remainders in both."""
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(h + w)
    disp = torch.from_numpy(rng.integers(0, 60, (B, h, w)).astype(np.uint8))
    img = torch.from_numpy(rng.integers(0, 256, (B, h, w)).astype(np.uint8))
    net = sv.TableVAE(f, dtype)
    es = ES[dtype]
    # weights the dtype holds exactly: the layer's own error is left
    params = torch.from_numpy(rng.normal(0, 0.1, net.nparams).astype(np.float32)).to(es).float()
    net.pack(params.cuda())
    net.forward(cuda(disp.numpy()), cuda(img.numpy()), h * f, w * f)
    torch.cuda.synchronize()
    l1 = net.workspace(B, h * f, w * f)[:B * h * w * 80 * es.itemsize].view(es).reshape(B, h, w, 80)
    got = l1[..., 16:].double().cpu().permute(0, 3, 1, 2)
    p = params.double()
    want, size = [], []
    for c, x in enumerate((disp.double() * f / 256, img.double() / 256)):
        wt, bias = p[c * 832:c * 832 + 800].reshape(32, 1, 5, 5), p[c * 832 + 800:c * 832 + 832]
        want.append(F.leaky_relu(F.conv2d(x[:, None], wt, bias, padding=2), 0.1))
        size.append(F.conv2d(x[:, None], wt.abs(), bias.abs(), padding=2))
    err = (got - torch.cat(want, 1)).abs()
    assert float((err / torch.cat(size, 1)).max()) <= FE_TOL[dtype] + (26 * 2.0 ** -24)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_infinities_of_the_map_and_weights_near_the_largest(dtype):
    """Where the map holds an infinity the output is what IEEE sums of w x give (the
    infinity, or NaN where two meet), and finite elsewhere; a finite weight beyond
    the largest BF16 value stays finite."""
    import paper_2305_11566_amd as sv
    rng = np.random.default_rng(31)
    f, h, w = 2, 40, 240
    H, W, es = h * f, w * f, ES[dtype]
    disp = np.zeros((1, h, w), np.uint8)
    disp[0, 3, 5] = disp[0, 20, 31] = 200
    img = rng.integers(0, 256, (1, h, w)).astype(np.uint8)
    # every weight positive: the layers below and D's part of the upsampling layer
    # keep infinities of one sign; its other weights have both signs
    params = rng.uniform(1e-3, 2e-3, sv.TableVAE(f, dtype).nparams).astype(np.float32)
    params[:25] = 3e38 if dtype != "f16" else 6e4  # FE_1's first output overflows where X_0 > 0
    params[-2026 + 16 * 25:] = rng.normal(0, 0.1, 2026 - 16 * 25)
    big = -2026 + 25 * 40 + 7                      # one weight of an FE_1 channel
    if dtype == "bf16":
        params[big] = 3.4e38
        params[16 * 25:32 * 25] = 0                # whose map (with its bias) is small
        params[800 + 16:832] = 1e-6
    net = sv.TableVAE(f, dtype)
    net.pack(cuda(params))
    out, _ = net.forward(cuda(disp), cuda(img), H, W)
    torch.cuda.synchronize()
    l1 = net.workspace(1, H, W)[:h * w * 80 * es.itemsize].view(es).reshape(1, h, w, 80)
    l1 = l1.double().cpu().permute(0, 3, 1, 2)
    assert torch.isinf(l1).any() and torch.isfinite(l1[..., -40:]).all() and not torch.isnan(l1).any()
    p = torch.from_numpy(params).double()
    x0 = torch.from_numpy(disp).double()[:, None] * f / 256
    cat = F.pad(torch.cat([l1[:, :16], x0, l1[:, 16:]], 1), (0, 2, 0, 2))
    want = 256 * (F.conv_transpose2d(cat, p[-2026:-1].reshape(81, 1, 5, 5), stride=f, padding=2)[:, 0, :H, :W] + p[-1])
    got = out.double().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isinf(got), torch.isinf(want))
    assert torch.isinf(want).any() and torch.isfinite(want).any()
    m = torch.isinf(want)
    assert torch.equal(got[m], want[m])
    m = torch.isfinite(want)
    assert float((got[m] - want[m]).abs().max() / want[m].abs().max()) <= TOL_F32
