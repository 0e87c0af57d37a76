"""The work that programs have this library do, as cases that can be timed.

`listed()` names them, `draw(rng)` gives more of the same ranges, `prepare`
makes what a program holds before the call (inputs from the seed, packed
weights, plans, captured graphs), `run` is one pass through the package's
public entry points, `work` the bytes and operations a pass cannot do without,
and `exact` what the pass returns in 64 bits, from plain torch alone.

The kinds of pass:
  match        reduction + census of both views, Hamming cost + winner-take-all
  sgm          the same with semi-global matching on the census or ZNCC cost,
               then the single matching phase and the median
  frame        a pair to its refined map: match, then the configurable network
  refine       that network alone on a coarse map a program already holds
  table        the Table I network alone
  train        matching, training forward, loss and gradients of the
               configurable network
  train_table  the same for the Table I network and its loss
  uneven       a batch of pairs of uneven sizes through one batch plan
"""
import math

import torch
import torch.nn.functional as F

import paper_2305_11566_amd as sv

SMALL = {"c1": 16, "c2": 32, "c3": 64, "latent": 64}     # the 256x128 network
LARGE = {"c1": 32, "c2": 64, "c3": 128, "latent": 128}   # the 1242x375 network
P1, P2 = 10, 120                                         # semi-global matching penalties
KL_WEIGHT = 1e-3
# (out, in, k) of the Table I network in parameter order
TABLE = [(32, 1, 5), (32, 1, 5), (16, 64, 5), (8, 16, 5), (32, 24, 5), (16, 32, 5), (2, 48, 1), (32, 1, 1),
         (16, 80, 5), (16, 96, 5), (8, 40, 5), (16, 48, 5), (1, 81, 5)]


def listed():
    kitti = {"H": 375, "W": 1242, "factor": 4, "win_w": 9, "win_h": 7, "D": 48}
    small = {"H": 128, "W": 256, "factor": 2, "win_w": 5, "win_h": 5, "D": 16}
    crop = {"H": 256, "W": 512, "factor": 2, "win_w": 5, "win_h": 5, "D": 16}
    return [
        # the smallest call: one small pair matched at once, as it arrives
        {"name": "match 256x128 b1", "kind": "match", "B": 1, **small},
        # a camera's frames one by one with the aggregating matcher, replayed from a graph
        {"name": "sgm census 1242x375 b1", "kind": "sgm", "matcher": "census", "graph": True, "B": 1, **kitti},
        # recorded sequences through the paper's main matcher
        {"name": "sgm zncc 1242x375 b16", "kind": "sgm", "matcher": "zncc", "graph": False, "B": 16, **kitti},
        # live frames: pair to refined map at batch 1, replayed from a graph
        {"name": "frame f32 1242x375 b1", "kind": "frame", "dtype": "f32", "graph": True, "B": 1, **kitti, **LARGE},
        # offline processing of recorded frames in large batches
        {"name": "frame bf16 1242x375 b64", "kind": "frame", "dtype": "bf16", "graph": False, "B": 64, **kitti,
         **LARGE},
        # a server that refines a few small coarse maps a call
        {"name": "refine f16 256x128 b8", "kind": "refine", "dtype": "f16", "B": 8, **small, **SMALL},
        # the quantised network on a few frames
        {"name": "refine i8 1242x375 b8", "kind": "refine", "dtype": "i8", "B": 8, **kitti, **LARGE},
        # the Table I network on live frames, replayed from a graph, and on batches
        {"name": "table f32 1242x375 b1", "kind": "table", "dtype": "f32", "graph": True, "B": 1, **kitti},
        {"name": "table bf16 1242x375 b16", "kind": "table", "dtype": "bf16", "graph": False, "B": 16, **kitti},
        # training on 512x256 crops, batch 16, and the Table I network's on a small batch
        {"name": "train bf16 512x256 b16", "kind": "train", "dtype": "bf16", "B": 16, **crop, **SMALL},
        {"name": "train table f32 512x256 b4", "kind": "train_table", "dtype": "f32", "B": 4, **crop},
        # a data set of uneven pairs, 64 a call
        {"name": "uneven bf16 n64", "kind": "uneven", "dtype": "bf16", "n": 64, "max_H": 384, "max_W": 1280,
         "factor": 4, "win_w": 9, "win_h": 7, "D": 80, "step": 8, **LARGE},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["match", "sgm", "frame", "refine", "table", "train", "train_table", "uneven"])
    if kind == "uneven":
        return {"kind": kind, "dtype": rng.choice(["f32", "bf16"]), "n": _log_int(rng, 2, 48),
                "max_H": rng.randint(128, 384), "max_W": rng.randint(320, 1280), "factor": 4, "win_w": 9, "win_h": 7,
                "D": rng.randint(24, 80), "step": rng.choice([1, 8]), **LARGE}
    H, W = _log_int(rng, 96, 400), _log_int(rng, 192, 1280)
    c = {"kind": kind, "H": H, "W": W}
    if kind in ("train", "train_table"):
        H, W = c["H"], c["W"] = _log_int(rng, 96, 280), _log_int(rng, 192, 560)
    if kind in ("train", "train_table") or W < 420:
        c.update(factor=2, win_w=5, win_h=5, D=rng.randint(12, 32))
    else:
        c.update(factor=4, win_w=9, win_h=7, D=rng.randint(24, 72))
    most = {"match": 64, "sgm": 24, "frame": 48, "refine": 48, "table": 32, "train": 16, "train_table": 8}[kind]
    B = _log_int(rng, 1, most)
    c["B"] = max(1, min(B, int(most * 375 * 1242 / 16 * c["factor"] ** 2 / (H * W))))
    if kind == "sgm":
        c["matcher"] = rng.choice(["census", "zncc"])
    if kind in ("sgm", "frame", "table"):
        c["graph"] = c["B"] <= 2
    if kind in ("frame", "refine"):
        c["dtype"] = rng.choice(["f32", "bf16", "bf16", "f16", "i8"])
    elif kind in ("table", "train", "train_table"):
        c["dtype"] = rng.choice(["f32", "bf16"])
    if kind in ("frame", "refine"):
        c.update(SMALL if c["factor"] == 2 else LARGE)
    elif kind == "train":
        c.update(SMALL)
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (salt + 1) + int(seed))
    return g


def _cdiv(a, b):
    return -(-a // b)


def _texture(g, B, H, W):
    """Blurred noise, the texture of natural surfaces, float [B, H, W] in 0..255."""
    x = torch.rand((B, 1, H + 10, W + 10), generator=g, device="cuda") * 255.0
    k = torch.exp(-0.5 * (torch.arange(-5.0, 6.0, device="cuda") / 1.5) ** 2)
    k = k / k.sum()
    x = sum(k[i] * x[:, :, i:i + H, :] for i in range(11))
    x = sum(k[i] * x[:, :, :, i:i + W] for i in range(11))
    return ((x[:, 0] - 127.5) * 4.0 + 127.5).clamp(0.0, 255.0)


def _planes(g, B, H, W, dmax):
    """Piecewise planar disparities in [0, dmax], float [B, H, W]: the nearest of 18 seeds gives the plane."""
    n = 18
    sy = torch.rand((B, n, 1, 1), generator=g, device="cuda") * H
    sx = torch.rand((B, n, 1, 1), generator=g, device="cuda") * W
    d0 = torch.rand((B, n, 1, 1), generator=g, device="cuda") * dmax
    sl = (torch.rand((B, n, 2), generator=g, device="cuda") - 0.5) * 0.1
    y = torch.arange(H, device="cuda", dtype=torch.float32).view(1, 1, H, 1)
    x = torch.arange(W, device="cuda", dtype=torch.float32).view(1, 1, 1, W)
    out = torch.empty((B, H, W), device="cuda")
    for b in range(B):
        dy, dx = y - sy[b], x - sx[b]
        near = (dy * dy + dx * dx).argmin(dim=1, keepdim=True)
        plane = d0[b] + sl[b, :, 0].view(1, n, 1, 1) * dy + sl[b, :, 1].view(1, n, 1, 1) * dx
        out[b] = plane.gather(1, near)[0, 0].clamp(0.0, dmax)
    return out


def _pairs(g, B, H, W, dmax):
    """(left, right uint8, disparity float) [B, H, W]: the right view samples the left one at x + d."""
    left = _texture(g, B, H, W).round()
    d = _planes(g, B, H, W, dmax)
    x = (torch.arange(W, device="cuda").view(1, 1, W) + d.round().long()).clamp(max=W - 1)
    right = left.gather(2, x) + 2.0 * torch.randn((B, H, W), generator=g, device="cuda")
    return left.to(torch.uint8), right.round().clamp(0, 255).to(torch.uint8), d


def _coarse(g, c):
    """A coarse disparity map with a matcher's outliers and a reduced left image, uint8 [B, h, w]."""
    B, h, w = c["B"], _cdiv(c["H"], c["factor"]), _cdiv(c["W"], c["factor"])
    d = _planes(g, B, h, w, c["D"] - 1.0).round()
    wild = torch.rand((B, h, w), generator=g, device="cuda") < 0.08
    d = torch.where(wild, torch.randint(0, c["D"], (B, h, w), generator=g, device="cuda").float(), d)
    return d.to(torch.uint8), _texture(g, B, h, w).round().to(torch.uint8)


def _refiner_shapes(c):
    c1, c2, c3, L = c["c1"], c["c2"], c["c3"], c["latent"]
    return [(c1, 2, 3), (c2, c1, 3), (c3, c2, 3), (2 * L, c3, 1), (c3, L, 1), (c2, c3 + c2, 3), (c1, c2 + c1, 3),
            (c1, c1 + 2, 3), (1, c1 + 2, 3)]


def _params(g, shapes, last):
    """He-normal weights and small biases as one FP32 vector; the last layer scaled by `last`, as training leaves it."""
    parts = []
    for i, (o, n, k) in enumerate(shapes):
        s = last if i == len(shapes) - 1 else 1.0
        parts.append(torch.randn(o * n * k * k, generator=g, device="cuda") * (s * math.sqrt(2.0 / (n * k * k))))
        parts.append((torch.rand(o, generator=g, device="cuda") - 0.5) * (0.2 * s))
    return torch.cat(parts)


def _layers(vec, shapes):
    out, at = [], 0
    for o, n, k in shapes:
        w = vec[at:at + o * n * k * k].view(o, n, k, k)
        at += o * n * k * k
        out.append((w, vec[at:at + o]))
        at += o
    return out


def _sizes(c):
    """(H, W, D) of the pairs of an uneven batch: half to all of the largest size, in steps of c["step"]."""
    at = torch.rand((c["n"], 2), generator=torch.Generator().manual_seed(c["n"])).tolist()
    cut = lambda most, r: int(most * (0.5 + 0.5 * r)) // c["step"] * c["step"]  # noqa: E731
    sizes = [(cut(c["max_H"], r), cut(c["max_W"], q)) for r, q in at]
    return [(H, W, max(8, c["D"] * W // c["max_W"])) for H, W in sizes]


def _inputs(c, seed):
    """All tensors of a case, from the seed alone."""
    g, kind = _gen(seed), c["kind"]
    if kind == "uneven":
        pairs = []
        for H, W, D in _sizes(c):
            left, right, _ = _pairs(g, 1, H, W, 4.0 * D - 2)
            pairs.append((left[0], right[0], D))
        return {"pairs": pairs, "params": _params(g, _refiner_shapes(c), 0.05)}
    if kind in ("refine", "table"):
        disp, low = _coarse(g, c)
        x = {"disp": disp, "low": low}
    else:
        left, right, d = _pairs(g, c["B"], c["H"], c["W"], c["factor"] * c["D"] - 2.0)
        x = {"left": left, "right": right, "gt": d}
    if kind in ("frame", "refine", "train"):
        x["params"] = _params(g, _refiner_shapes(c), 0.05)
    elif kind in ("table", "train_table"):
        x["params"] = _params(g, TABLE, 1.0)
    if kind == "train":
        h, w = _cdiv(c["H"], 8 * c["factor"]), _cdiv(c["W"], 8 * c["factor"])
        x["eps"] = torch.randn((c["B"], h, w, c["latent"]), generator=g, device="cuda")
    elif kind == "train_table":
        h, w = _cdiv(c["H"], 4 * c["factor"]), _cdiv(c["W"], 4 * c["factor"])
        x["eps"] = torch.randn((c["B"], h, w), generator=g, device="cuda")
        occ = torch.rand(d.shape, generator=g, device="cuda") < 0.95
        x["occ"] = occ.to(torch.uint8)
        x["noc"] = (occ & (torch.rand(d.shape, generator=g, device="cuda") < 0.9)).to(torch.uint8)
    return x


# ------------------------------------------------------------------ the passes

def _match(s):
    c, out = s["case"], s["match_out"]
    cl, cr, low = sv.sv_census_pair(s["left"], s["right"], c["factor"], c["win_w"], c["win_h"], out=out and out[:3])
    disp = sv.sv_cost_wta(cl, cr, c["D"], c["win_w"] * c["win_h"] - 1, out=out and out[3])
    return cl, cr, low, disp


def _pass(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "match":
        cl, cr, low, disp = _match(s)
        return {"census_left": cl, "census_right": cr, "reduced": low, "disparity": disp}
    if kind == "sgm":
        cl, cr, low, low_r = s["census"]
        if c["matcher"] == "census":
            sv.sv_census_pair(s["left"], s["right"], c["factor"], c["win_w"], c["win_h"], out=(cl, cr, low))
            raw = sv.sv_sgm(cl, cr, c["D"], c["win_w"] * c["win_h"] - 1, P1, P2, out=s["raw"], workspace=s["sgm_ws"])
        else:
            sv.sv_census(s["left"], c["factor"], c["win_w"], c["win_h"], out=(cl, low))
            sv.sv_census(s["right"], c["factor"], c["win_w"], c["win_h"], out=(cr, low_r))
            raw = sv.sv_zncc_sgm(low, low_r, c["D"], c["win_w"], c["win_h"], P1, P2, out=s["raw"],
                                 workspace=s["sgm_ws"])
        return {"aggregated": raw, "disparity": sv.sv_smp_median(raw, c["D"], out=s["disp"], workspace=s["smp_ws"]),
                "reduced": low}
    if kind in ("frame", "refine"):
        disp, low = s.get("disp"), s.get("low")
        if kind == "frame":
            _, _, low, disp = _match(s)
        out, ml = s["net"].forward(disp, low, c["H"], c["W"], out=s["out"], mu_logvar=s["latent_out"])
        return {"disparity": disp, "refined": out, "mu_logvar": ml}
    if kind == "table":
        out, ms = s["net"].forward(s["disp"], s["low"], c["H"], c["W"], out=s["out"], mu_sigma=s["latent_out"])
        return {"refined": out, "mu_sigma": ms}
    if kind == "train":
        net, B, H, W = s["net"], c["B"], c["H"], c["W"]
        net.pack(s["params"])
        _, _, low, disp = _match(s)
        out, ml = net.forward(disp, low, H, W, eps=s["eps"], saved=s["saved"])
        loss, dout = sv.sv_loss(out, s["gt"], ml, c["latent"], KL_WEIGHT)
        grad = net.backward(s["saved"], B, H, W, s["eps"], dout, KL_WEIGHT)
        return {"refined": out, "mu_logvar": ml, "loss": loss, "grad": grad}
    if kind == "train_table":
        net, H, W = s["net"], c["H"], c["W"]
        net.pack(s["params"])
        _, _, low, disp = _match(s)
        out, ms = net.forward(disp, low, H, W, eps=s["eps"])
        loss, dout, dms = sv.sv_tvae_loss(out, s["gt"], s["noc"], s["occ"], ms)
        grad = net.backward(disp, low, H, W, dout, eps=s["eps"], dmu_sigma=dms)
        return {"refined": out, "mu_sigma": ms, "loss": loss, "grad": grad}
    return s["plan"].run(s["pairs"], s["net"].packed, outs=s["outs"])


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "match_out": None, **_inputs(c, seed)}
    if kind in ("sgm", "frame"):
        B, h, w = c["B"], _cdiv(c["H"], c["factor"]), _cdiv(c["W"], c["factor"])
        word = [torch.empty((B, h, w), dtype=torch.int64, device="cuda") for _ in range(2)]
        byte = [torch.empty((B, h, w), dtype=torch.uint8, device="cuda") for _ in range(4)]
        s["census"] = (*word, byte[0], byte[1])
        s["match_out"] = (*word, byte[0], byte[1])
        if kind == "sgm":
            s["raw"], s["disp"] = byte[2], byte[3]
            s["sgm_ws"] = torch.empty(sv.lib().sv_sgm_workspace_bytes(B, h, w, c["D"]), dtype=torch.uint8,
                                      device="cuda")
            s["smp_ws"] = torch.empty(sv.lib().sv_smp_workspace_bytes(B, h, w), dtype=torch.uint8, device="cuda")
    if kind in ("frame", "refine", "train", "uneven"):
        s["net"] = sv.Refiner(c["c1"], c["c2"], c["c3"], c["latent"], c["factor"], c["dtype"])
        s["net"].pack(s["params"])
    elif kind in ("table", "train_table"):
        s["net"] = sv.TableVAE(c["factor"], c["dtype"])
        s["net"].pack(s["params"])
    if kind in ("frame", "refine", "table"):
        net, B, H, W = s["net"], c["B"], c["H"], c["W"]
        s["out"] = torch.empty((B, H, W), dtype=torch.float32, device="cuda")
        shape = net.latent_shape(B, H, W)
        shape = shape + (2,) if kind == "table" else shape[:3] + (2 * c["latent"],)
        s["latent_out"] = torch.empty(shape, dtype=torch.float32, device="cuda")
        net.workspace(B, H, W)
    if kind in ("train", "train_table"):
        s["net"].workspace(c["B"], c["H"], c["W"])
    if kind == "train":
        s["saved"] = s["net"].saved_buffer(c["B"], c["H"], c["W"])
    if kind == "uneven":
        s["plan"] = sv.BatchPlan(c["c1"], c["c2"], c["c3"], c["latent"], c["factor"], c["dtype"], c["n"], c["max_H"],
                                 c["max_W"], c["D"], c["win_w"], c["win_h"])
        s["outs"] = [torch.empty(left.shape, dtype=torch.float32, device="cuda") for left, _, _ in s["pairs"]]
    if c.get("graph"):
        _pass(s)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["graph_out"] = _pass(s)
    return s


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["graph_out"]
    return _pass(state)


# ------------------------------------------------------------------ what a pass cannot do without

def _levels(c, H, W, n):
    hw = [(_cdiv(H, c["factor"]), _cdiv(W, c["factor"]))]
    for _ in range(n - 1):
        hw.append((_cdiv(hw[-1][0], 2), _cdiv(hw[-1][1], 2)))
    return [h * w for h, w in hw]


def _refiner_macs(c, H, W):
    p = _levels(c, H, W, 4)
    s = [o * n * k * k for o, n, k in _refiner_shapes(c)]
    # the final layer as nine projections at the coarse level, four corners of nine taps each gathered
    return (p[1] * s[0] + p[2] * s[1] + p[3] * (s[2] + s[3] + s[4]) + p[2] * s[5] + p[1] * s[6] + p[0] * (s[7] + s[8])
            + H * W * 9)


def _table_macs(c, H, W):
    p = _levels(c, H, W, 3)
    s = [o * n * k * k for o, n, k in TABLE]
    return (p[0] * (s[0] + s[1] + s[12]) + p[1] * (s[2] + s[3] + s[10] + s[11])
            + p[2] * (s[4] + s[5] + s[6] + s[7] + s[8] + s[9]))


def work(case):
    c, kind = case, case["kind"]
    if kind == "uneven":
        ops = nbytes = 0
        for H, W, D in _sizes(c):
            ops += 2 * _refiner_macs(c, H, W) + _levels(c, H, W, 1)[0] * 6 * D
            nbytes += 6 * H * W
        return {"bytes": nbytes + 4 * sum(o * n * k * k + o for o, n, k in _refiner_shapes(c)), "flops": ops}
    B, H, W = c["B"], c["H"], c["W"]
    px = B * _levels(c, H, W, 1)[0]
    full = B * H * W
    hamming = 6 * px * c["D"]             # exclusive or, popcount (two halves), pack, minimum
    if kind == "match":
        return {"bytes": 2 * full + (16 + 2) * px, "flops": hamming}
    if kind == "sgm":
        taps = c["win_w"] * c["win_h"]
        cost = hamming if c["matcher"] == "census" else 2 * taps * px * c["D"]
        return {"bytes": 2 * full + 3 * px, "flops": cost + 4 * 8 * px * c["D"]}
    shapes = TABLE if kind in ("table", "train_table") else _refiner_shapes(c)
    macs = B * (_table_macs if kind in ("table", "train_table") else _refiner_macs)(c, H, W)
    nbytes = 4 * sum(o * n * k * k + o for o, n, k in shapes) + 4 * full
    if kind in ("refine", "table"):
        return {"bytes": nbytes + 2 * px, "flops": 2 * macs}
    if kind == "frame":
        return {"bytes": nbytes + 2 * full + px, "flops": 2 * macs + hamming}
    # forward, the gradient of the inputs and that of the weights
    return {"bytes": 2 * nbytes + 6 * full, "flops": 6 * macs + hamming}


# ------------------------------------------------------------------ the same in 64 bits

def _conv64(x, w, b, stride=1):
    """NHWC convolution, padding (k - 1) / 2, as a sum of one matrix product a tap."""
    k = w.shape[-1]
    p = (k - 1) // 2
    B, H, W, C = x.shape
    h, v = (H + 2 * p - k) // stride + 1, (W + 2 * p - k) // stride + 1
    xp = F.pad(x, (0, 0, p, p, p, p))
    y = b.expand(B * h * v, -1)
    for i in range(k):
        for j in range(k):
            t = xp[:, i:i + stride * (h - 1) + 1:stride, j:j + stride * (v - 1) + 1:stride, :]
            y = y + t.reshape(-1, C) @ w[:, :, i, j].t()
    return y.view(B, h, v, -1)


def _deconv64(x, w, b, stride, H, W):
    """NHWC transposed convolution, padding (k - 1) / 2, cut to H x W."""
    k = w.shape[-1]
    p = (k - 1) // 2
    B, h, v, C = x.shape
    full = x.new_zeros((B, max(stride * (h - 1) + k, H + p), max(stride * (v - 1) + k, W + p), w.shape[0]))
    for i in range(k):
        for j in range(k):
            t = (x.reshape(-1, C) @ w[:, :, i, j].t()).view(B, h, v, -1)
            full[:, i:i + stride * (h - 1) + 1:stride, j:j + stride * (v - 1) + 1:stride, :] += t
    return full[:, p:p + H, p:p + W, :] + b


def _resize64(x, H, W):
    return F.interpolate(x.permute(0, 3, 1, 2), size=(H, W), mode="bilinear", align_corners=False).permute(0, 2, 3, 1)


def _refine64(c, params, disp, low, H, W, eps=None):
    """-> (refined map [B, H, W], mu and log-variance [B, h, w, 2 L])."""
    p = _layers(params, _refiner_shapes(c))
    act = lambda x: F.leaky_relu(x, 0.1)  # noqa: E731
    x0 = torch.stack([c["factor"] * disp.double() / 256.0, low.double() / 256.0], dim=3)
    e1 = act(_conv64(x0, *p[0], 2))
    e2 = act(_conv64(e1, *p[1], 2))
    e3 = act(_conv64(e2, *p[2], 2))
    ml = _conv64(e3, *p[3])
    mu, lv = ml[..., :c["latent"]], ml[..., c["latent"]:]
    g = act(_conv64(mu if eps is None else mu + eps.double() * torch.exp(0.5 * lv), *p[4]))
    for i, skip in ((5, e2), (6, e1), (7, x0)):
        g = act(_conv64(torch.cat([_resize64(g, skip.shape[1], skip.shape[2]), skip], dim=3), *p[i]))
    r = _conv64(_resize64(torch.cat([g, x0], dim=3), H, W), *p[8])[..., 0]
    return 256.0 * (r + _resize64(x0[..., :1], H, W)[..., 0]), ml


def _table64(c, params, disp, low, H, W, eps=None):
    """-> (refined map [B, H, W], mu and sigma [B, h, w, 2])."""
    p = _layers(params, TABLE)
    act = lambda x: F.leaky_relu(x, 0.1)  # noqa: E731
    cat = lambda *x: torch.cat(x, dim=3)  # noqa: E731
    x0, x1 = c["factor"] * disp.double()[..., None] / 256.0, low.double()[..., None] / 256.0
    fe = cat(act(_conv64(x0, *p[0])), act(_conv64(x1, *p[1])))
    en1 = act(_conv64(fe, *p[2], 2))
    en1 = cat(en1, act(_conv64(en1, *p[3])))
    en2 = act(_conv64(en1, *p[4], 2))
    en2 = cat(en2, act(_conv64(en2, *p[5])))
    ms = _conv64(en2, *p[6])
    z = ms[..., :1] - 1.0
    if eps is not None:
        z = z + eps.double()[..., None] * torch.exp(ms[..., 1:] - 1.0)
    d1 = cat(act(_conv64(z, *p[7])), en2)
    d1 = cat(d1, act(_conv64(d1, *p[8])))
    d2 = cat(act(_deconv64(d1, *p[9], 2, en1.shape[1], en1.shape[2])), en1)
    d2 = cat(d2, act(_conv64(d2, *p[10])))
    d = act(_deconv64(d2, *p[11], 2, fe.shape[1], fe.shape[2]))
    y = _deconv64(cat(d, x0, fe), *p[12], c["factor"], H, W)
    return 256.0 * y[..., 0], ms


def _reduced(img, f):
    """f x f block means, rounded half up, partial blocks over their own pixels."""
    x = img.long()[:, None]
    H, W = img.shape[1:]
    pad = (0, -W % f, 0, -H % f)
    s = F.pad(x, pad).unfold(2, f, f).unfold(3, f, f).sum(dim=(4, 5))
    n = F.pad(torch.ones_like(x[:1]), pad).unfold(2, f, f).unfold(3, f, f).sum(dim=(4, 5))
    return ((2 * s + n) // (2 * n))[:, 0]


def _census_bits(low, ww, wh):
    """bool [bits, B, h, w]: whether each neighbour is darker, borders clamped."""
    h, w = low.shape[1:]
    p = F.pad(low[:, None].float(), (ww // 2, ww // 2, wh // 2, wh // 2), mode="replicate")[:, 0]
    return torch.stack([p[:, i:i + h, j:j + w] < low for i in range(wh) for j in range(ww)
                        if (i, j) != (wh // 2, ww // 2)])


def _coarse64(c, left, right, D):
    """-> (disparity, reduced left image), one pair at a time."""
    disp, lows = [], []
    for k in range(left.shape[0]):
        ll, lr = _reduced(left[k:k + 1], c["factor"]), _reduced(right[k:k + 1], c["factor"])
        bl, br = _census_bits(ll, c["win_w"], c["win_h"]), _census_bits(lr, c["win_w"], c["win_h"])
        w = ll.shape[2]
        cost = torch.full((D, *ll.shape), bl.shape[0] + 1, device="cuda", dtype=torch.long)
        for d in range(min(D, w)):
            cost[d, :, :, d:] = (bl[..., d:] ^ br[..., :w - d]).sum(dim=0)
        disp.append((cost * 256 + torch.arange(D, device="cuda").view(D, 1, 1, 1)).amin(dim=0) % 256)
        lows.append(ll)
    return torch.cat(disp), torch.cat(lows)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("match", "sgm"):
        return None  # whole numbers alone
    x = _inputs(c, seed)
    params = x["params"].double()
    if kind == "uneven":
        outs = []
        for left, right, D in x["pairs"]:
            disp, low = _coarse64(c, left[None], right[None], D)
            outs.append(_refine64(c, params, disp, low, *left.shape)[0][0])
        return outs
    H, W = c["H"], c["W"]
    if kind in ("refine", "table"):
        disp, low = x["disp"], x["low"]
    else:
        disp, low = _coarse64(c, x["left"], x["right"], c["D"])
    if kind in ("frame", "refine", "table"):
        # the quantised network is held against the one it stands for
        net = _table64 if kind == "table" else _refine64
        parts = [net(c, params, disp[k:k + 4], low[k:k + 4], H, W) for k in range(0, c["B"], 4)]
        out, lat = (torch.cat([p[i] for p in parts]) for i in range(2))
        if kind == "table":
            return {"refined": out, "mu_sigma": lat}
        return {"disparity": None, "refined": out, "mu_logvar": lat}
    params.requires_grad_(True)
    if kind == "train":
        out, ml = _refine64(c, params, disp, low, H, W, x["eps"])
        mu, lv = ml[..., :c["latent"]], ml[..., c["latent"]:]
        data = F.smooth_l1_loss(out, x["gt"].double())
        kl = (0.5 * (mu ** 2 + torch.exp(lv) - 1.0 - lv)).mean()
        total, latent = data + KL_WEIGHT * kl, "mu_logvar"
    else:
        out, ml = _table64(c, params, disp, low, H, W, x["eps"])
        mu, sg = ml[..., 0] - 1.0, ml[..., 1] - 1.0
        err, noc, occ = (out - x["gt"].double()).abs(), x["noc"].double(), x["occ"].double()
        data = (err * (noc + occ)).sum() / occ.sum()
        kl = 256.0 * (0.5 * (mu ** 2 - 1.0 + torch.exp(2.0 * sg) - 2.0 * sg)).mean()
        total, latent = data + kl, "mu_sigma"
    total.backward()
    return {"refined": out.detach(), latent: ml.detach(), "loss": torch.stack([total, data, kl]).detach(),
            "grad": params.grad}
