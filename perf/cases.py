"""The measured cases: batched total-variation proximal operators as a program calls them.

A case is one call, or one forward and backward pair, through the package's public entry points:

  path       "rows"   1D along the last axis of [B, C, H, W] (a batch of plain rows is [1, R, 1, n])
             "cols"   1D along H
             "planes" 2D with `sweeps` iterations
  direction  "infer" (forward), "train" (forward, then backward from what the forward call left) or
             "backward" (the backward call alone, on a solution that the program already holds)
  api        "abi" (the ctypes binding, buffers owned by the caller) or "layer" (TVLayer and autograd)
  data       "maps" N(0,1) feature maps; "relu" the same behind a ReLU (half zeros, many ties);
             "steps" constant segments plus noise; "walk" a random walk with jumps;
             "image" piecewise-smooth images plus noise
  lam        "scalar", "channel" or "row": one lambda, one a channel, one a row;
             lam_lo .. lam_hi its range (log-uniform)
  dtype      "f32" or "bf16" (storage; where the package has it: 2D planes of at most 32 x 32)
"""
import math

import torch

import paper_2204_03643_amd as tv
from paper_2204_03643_amd.layer import TVLayer


def _case(name, path, direction, api, B, C, H, W, data, lam, lam_lo, lam_hi, sweeps=0, dtype="f32"):
    c = dict(path=path, direction=direction, api=api, B=B, C=C, H=H, W=W, data=data, lam=lam,
             lam_lo=lam_lo, lam_hi=lam_hi, sweeps=sweeps, dtype=dtype)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a handful of signals denoised and differentiated in an interactive loop: launch latency
        _case("rows_64x256_train", "rows", "train", "abi", 1, 64, 1, 256, "steps", "scalar", 0.5, 0.5),
        # the batch of the paper's timing table: 8192 noisy steps of 32 samples
        _case("rows_8192x32_train", "rows", "train", "abi", 1, 8192, 1, 32, "steps", "scalar", 1.0, 1.0),
        # one training step's 1D layer on a large batch of 32 x 32 feature maps (the benchmark's headline)
        _case("maps_256x128x32x32_rows_train", "rows", "train", "abi", 256, 128, 32, 32, "maps", "channel", 1e-3, 10.0),
        # the backward call of a 1D layer along the columns of images, on a solution from earlier
        _case("image_8x3x512x512_cols_backward", "cols", "backward", "abi", 8, 3, 512, 512, "image", "scalar", 0.1, 0.1),
        # the paper's TV layer on a small batch of feature maps, through autograd
        _case("layer_4x64x32x32_k4_train", "planes", "train", "layer", 4, 64, 32, 32, "maps", "channel", 0.05, 1.0, 4),
        # the same layer on a larger batch kept in bf16
        _case("layer_64x64x32x32_k3_bf16_train", "planes", "train", "layer", 64, 64, 32, 32, "maps", "channel", 0.05, 1.0, 3, "bf16"),
        # planes that fill no power of two, in inference behind a ReLU
        _case("maps_51x105x28x28_k4_infer", "planes", "infer", "abi", 51, 105, 28, 28, "relu", "channel", 0.01, 1.0, 4),
        # feature maps of an early layer
        _case("maps_16x64x64x64_k4_train", "planes", "train", "abi", 16, 64, 64, 64, "maps", "channel", 0.05, 1.0, 4),
        # colour images denoised with ten sweeps, with gradients
        _case("image_8x3x512x512_k10_train", "planes", "train", "abi", 8, 3, 512, 512, "image", "scalar", 0.1, 0.1, 10),
        # photographs of odd size, denoised only
        _case("image_4x3x321x481_k3_infer", "planes", "infer", "layer", 4, 3, 321, 481, "image", "channel", 0.03, 0.3, 3),
        # ragged long signals, a lambda for each
        _case("rows_2999x3001_infer", "rows", "infer", "abi", 1, 2999, 1, 3001, "steps", "row", 1e-3, 10.0),
        # the longest signals, with gradients
        _case("rows_4096x16384_train", "rows", "train", "abi", 1, 4096, 1, 16384, "walk", "row", 1e-3, 10.0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["rows", "rows", "cols", "planes", "planes"])
    direction = rng.choice(["infer", "train", "train", "backward"] if path != "planes" else ["infer", "train"])
    api = rng.choice(["abi", "abi", "layer"]) if direction != "backward" else "abi"
    total = math.exp(rng.uniform(math.log(1 << 14), math.log(1 << 25)))
    sweeps, dtype = 0, "f32"
    if path == "rows":
        n = 32 if rng.random() < 0.25 else _log_int(rng, 8, 16384)
        H = rng.choice([1, 1, n]) if n <= 512 else 1
        C = _log_int(rng, 1, 256) if H > 1 else 1
        rows = max(4, int(total / n))
        B, C, H, W = (max(1, rows // (C * H)), C, H, n) if H > 1 else (1, rows, 1, n)
        if api == "layer" and H == 1:
            C, H = 1, C                    # a batch of rows handed to the layer as one channel
    else:
        lo, hi = (8, 1024) if path == "cols" else (7, 768)
        H = 32 if rng.random() < 0.3 else _log_int(rng, lo, hi)
        W = H if rng.random() < 0.6 else max(lo, min(hi, int(H * rng.uniform(0.5, 2.0))))
        C = 3 if H * W > 100 * 100 else _log_int(rng, 8, 128)
        B = max(1, min(4096, int(total / (C * H * W))))
    if path == "planes":
        sweeps = rng.choice([1, 2, 3, 4, 4, 10])
        B = max(1, min(B, int((1 << 27) / (C * H * W * sweeps))))
        if max(H, W) <= 32 and rng.random() < 0.3:
            dtype = "bf16"
    n = H if path == "cols" else W
    if path != "rows" or H > 1:
        data = "image" if H * W > 100 * 100 else ("maps" if direction != "infer" else rng.choice(["maps", "relu"]))
    else:
        data = rng.choice(["steps", "walk"]) if n > 64 else rng.choice(["steps", "maps"])
    if data == "image":
        lam, lo, hi = rng.choice(["scalar", "channel"]), 0.03, 0.3
    elif path == "rows" and H == 1 and api == "abi":
        lam, lo, hi = rng.choice(["scalar", "row"]), 1e-3, 10.0
    else:
        lam, lo, hi = "channel", 0.01, 3.0
    if lam == "scalar":
        lo = hi = round(math.exp(rng.uniform(math.log(0.05), math.log(1.0))), 4)
    return _case(None, path, direction, api, B, C, H, W, data, lam, lo, hi, sweeps, dtype)


# ------------------------------------------------------------------------------------ inputs

def _signal(c, gen, dev):
    B, C, H, W = c["B"], c["C"], c["H"], c["W"]
    shape = (B, C, H, W)
    if c["data"] in ("maps", "relu"):
        y = torch.randn(shape, generator=gen, device=dev)
        return y.relu_() if c["data"] == "relu" else y
    if c["data"] == "walk":
        y = torch.randn(shape, generator=gen, device=dev).mul_(0.05)
        at = torch.rand(shape, generator=gen, device=dev)
        jump = torch.rand(shape, generator=gen, device=dev).mul_(1.5).add_(0.5)
        y += torch.where(at < 5e-4, jump, torch.where(at > 1 - 5e-4, -jump, torch.zeros_like(jump)))
        return y.cumsum_(-1)
    if c["data"] == "steps":               # eight segments a row or so, levels U(-1, 1), noise 0.1 .. 0.5
        at = torch.rand(shape, generator=gen, device=dev) < min(0.25, 8.0 / W)
        level = torch.rand(shape, generator=gen, device=dev).mul_(2).sub_(1)
        where = torch.arange(W, device=dev).expand(shape)
        last = torch.where(at, where, torch.zeros_like(where)).cummax(-1).values
        noise = torch.rand((B, C, 1, 1), generator=gen, device=dev).mul_(0.4).add_(0.1)
        return level.gather(-1, last) + noise * torch.randn(shape, generator=gen, device=dev)
    py = ((torch.arange(H, device=dev) + 0.5) / H).view(1, 1, H, 1)
    px = ((torch.arange(W, device=dev) + 0.5) / W).view(1, 1, 1, W)

    def ramp():
        k = torch.rand((3, B, C, 1, 1), generator=gen, device=dev)
        return k[0] + (k[1] - 0.5) * (px - 0.5) + (k[2] - 0.5) * (py - 0.5)

    img = ramp()
    for _ in range(12):                    # rotated rectangles, each with a ramp of its own
        k = torch.rand((5, B, 1, 1, 1), generator=gen, device=dev)
        cx, cy, a = px - 0.1 - 0.8 * k[0], py - 0.1 - 0.8 * k[1], 3.1416 * k[2]
        inside = ((cx * a.cos() + cy * a.sin()).abs() < 0.03 + 0.27 * k[3]) & ((cy * a.cos() - cx * a.sin()).abs() < 0.03 + 0.27 * k[4])
        img = torch.where(inside, ramp(), img)
    return img.clamp_(0, 1) + (25.0 / 255.0) * torch.randn(shape, generator=gen, device=dev)


def _inputs(c, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    y = _signal(c, gen, dev)
    B, C, H, W = y.shape
    count = {"scalar": 1, "channel": C, "row": B * C * H}[c["lam"]]
    lo, hi = math.log(c["lam_lo"]), math.log(c["lam_hi"])
    lam = torch.rand(count, generator=gen, device=dev).mul_(hi - lo).add_(lo).exp_()
    # the upstream gradient has a value of its own for each plane, as behind a pooled head, and a
    # part of its own for each sample
    g = torch.rand((B, C, 1 if H > 1 and W > 1 else H, 1), generator=gen, device=dev).add_(0.5)
    g = g + 0.2 * torch.randn(y.shape, generator=gen, device=dev)
    if c["dtype"] == "bf16":
        y, g = y.bfloat16(), g.bfloat16()
    return y, lam, g


def _solution(c, seed):
    """A piecewise-constant x as a forward call leaves it: segments of one sample up to about 64."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) + 77)
    shape = (c["B"], c["C"], c["H"], c["W"])
    axis = -2 if c["path"] == "cols" else -1
    p = torch.rand((c["B"], c["C"], 1, 1), generator=gen, device=dev).mul_(4.0).neg_().exp_()
    at = torch.rand(shape, generator=gen, device=dev) < p
    level = torch.randn(shape, generator=gen, device=dev)
    n = shape[axis]
    where = torch.arange(n, device=dev).view((n, 1) if axis == -2 else (n,)).expand(shape)
    last = torch.where(at, where, torch.zeros_like(where)).cummax(axis).values
    return level.gather(axis, last)


def _layer(c, lam):
    mode = {"rows": "rows", "cols": "cols", "planes": "2d"}[c["path"]]
    layer = TVLayer(c["C"], mode=mode, shared_lambda=c["lam"] == "scalar", sweeps=max(1, c["sweeps"])).cuda()
    with torch.no_grad():
        layer.raw_lambda.copy_(torch.log(torch.expm1(lam)))        # lambda = SoftPlus(parameter)
    return layer


class _Lines:
    """What a program keeps for 1D calls: the descriptors and the buffers."""

    def __init__(self, c, y, lam, g):
        B, C, H, W = y.shape
        self.rows = tv.rows_along(tuple(y.shape), -2 if c["path"] == "cols" else -1)
        div = {"scalar": 1, "row": 1, "channel": W if c["path"] == "cols" else H}[c["lam"]]
        self.lam = tv.tv_lambda(lam.data_ptr(), lam.numel(), div)
        self.y, self.lam_tensor, self.g = y, lam, g
        self.x, self.gy, self.gl = torch.empty_like(y), torch.empty_like(y), torch.empty_like(lam)
        self.seg = None
        if self.rows.length <= 32:
            self.seg = torch.empty(self.rows.n_outer * self.rows.n_inner, dtype=torch.int64, device=y.device)
        self.ws_bytes = tv.tv1d_bwd_workspace_bytes(self.rows, self.lam)
        self.ws = torch.empty(max(16, self.ws_bytes), dtype=torch.uint8, device=y.device)

    def forward(self):
        if self.seg is None:
            tv.tv1d_prox_fwd(self.y, self.x, self.rows, self.lam)
        else:
            tv.tv1d_prox_fwd_ex(self.y, self.x, self.rows, self.lam, seg=self.seg)

    def backward(self, plain=False):
        if self.seg is None or plain:
            tv.tv1d_prox_bwd(self.g, self.x, self.gy, self.gl, self.rows, self.lam, self.ws, self.ws_bytes)
        else:
            tv.tv1d_prox_bwd_seg(self.g, self.seg, self.gy, self.gl, self.rows, self.lam, self.ws, self.ws_bytes)


class _Planes:
    """The same for 2D calls."""

    def __init__(self, c, y, lam, g):
        B, C, self.H, self.W = y.shape
        self.planes, self.sweeps = B * C, c["sweeps"]
        self.lam = tv.tv_lambda(lam.data_ptr(), lam.numel(), 1)
        self.y, self.lam_tensor, self.g = y, lam, g
        self.x, self.gy, self.gl = torch.empty_like(y), torch.empty_like(y), torch.empty_like(lam)
        self.ws_bytes = tv.tv2d_workspace_bytes(self.planes, self.H, self.W, self.sweeps)
        self.ws = torch.empty(max(16, self.ws_bytes), dtype=torch.uint8, device=y.device)
        self.fwd = tv.tv2d_prox_fwd_bf16 if c["dtype"] == "bf16" else tv.tv2d_prox_fwd
        self.bwd = tv.tv2d_prox_bwd_bf16 if c["dtype"] == "bf16" else tv.tv2d_prox_bwd

    def forward(self):
        self.fwd(self.y, self.x, self.planes, self.H, self.W, self.lam, self.sweeps, self.ws, self.ws_bytes)

    def backward(self):
        self.bwd(self.g, self.gy, self.gl, self.planes, self.H, self.W, self.lam, self.sweeps, self.ws, self.ws_bytes)


def prepare(case, seed):
    y, lam, g = _inputs(case, seed)
    if case["api"] == "layer":
        return {"case": case, "y": y.requires_grad_(case["direction"] == "train"), "g": g, "layer": _layer(case, lam)}
    held = (_Planes if case["path"] == "planes" else _Lines)(case, y, lam, g)
    if case["direction"] == "backward":
        held.x.copy_(_solution(case, seed))
    return {"case": case, "held": held}


def run(state):
    direction = state["case"]["direction"]
    if "layer" in state:
        layer, y = state["layer"], state["y"]
        if direction == "infer":
            with torch.no_grad():
                return {"x": layer(y)}
        x = layer(y)
        gy, gl = torch.autograd.grad(x, [y, layer.raw_lambda], state["g"])
        return {"x": x.detach(), "grad_y": gy, "grad_lam": gl}
    held = state["held"]
    if direction == "backward":
        held.backward(plain=True)
        return {"grad_y": held.gy, "grad_lam": held.gl}
    held.forward()
    if direction == "infer":
        return {"x": held.x}
    held.backward()
    return {"x": held.x, "grad_y": held.gy, "grad_lam": held.gl}


# ---------------------------------------------------------------------------------- the floor

def work(case):
    samples = case["B"] * case["C"] * case["H"] * case["W"]
    size = 2 if case["dtype"] == "bf16" else 4
    passes = max(1, 2 * case["sweeps"])
    # forward: y in, x out; backward: g (and x, where the call gets nothing else) in, grad_y out.
    # One solve of a row is at least one elimination and one back substitution, its backward a sum
    # and a mean for each sample.
    tensors = {"infer": 2, "train": 4, "backward": 3}[case["direction"]]
    flops = {"infer": 20, "train": 26, "backward": 6}[case["direction"]]
    return {"bytes": float(tensors * size * samples), "flops": float(flops * passes * samples)}


def tolerance(case):
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.99}
    if case["direction"] == "train":
        # Where two neighbouring levels of x agree to rounding, the gradient's two segments are one
        # or two by the last bit of x: a few rows in a million, whole segments of them.
        return {"rel": 1e-2, "max": 0.99}
    if case["direction"] == "backward":
        return {"rel": 4e-6, "max": 2e-4}
    return {"rel": 1e-5, "max": 1e-3}


# ------------------------------------------------------------------------- the same in 64 bits

def _blocks(x, held):
    """Mean of x over the blocks that the held duals cut each row into, for every sample."""
    first = torch.ones_like(x, dtype=torch.bool)
    first[:, 1:] = held
    ids = first.reshape(-1).cumsum(0).sub_(1)
    count = int(ids[-1]) + 1
    flat = x.reshape(-1)
    size = torch.zeros(count, dtype=x.dtype, device=x.device).index_add_(0, ids, torch.ones_like(flat))
    mean = torch.zeros(count, dtype=x.dtype, device=x.device).index_add_(0, ids, flat).div_(size)
    return mean[ids].view_as(x)


def _primal(y, u):
    x = y.clone()
    x[:, :-1] += u
    x[:, 1:] -= u
    return x


def _prox64(y, lam):
    """Rows of y [R, n] with lam [R, 1], in 64 bits: projected Newton on the dual."""
    R, n = y.shape
    if n == 1:
        return y.clone()
    out = torch.empty_like(y)
    run = (y.mean(1, keepdim=True) - y).cumsum(1)[:, :-1]
    lam = torch.minimum(lam, 2 * run.abs().amax(1, keepdim=True))
    u = torch.where(lam >= 0.5 * run.abs().amax(1, keepdim=True), run.clamp(-lam, lam), lam * (y[:, 1:] - y[:, :-1]).sign())
    del run
    left = torch.arange(R, device=y.device)
    floor = 1e-13 * (y.abs().amax(1, keepdim=True) + lam)
    for _ in range(1000):
        x = _primal(y, u)
        f = 0.5 * x.square().sum(1, keepdim=True)
        g = x[:, :-1] - x[:, 1:]
        held = ((u <= -lam) & (g > 0)) | ((u >= lam) & (g < 0))
        inward = (((u <= -lam) & (g < -floor)) | ((u >= lam) & (g > floor))).any(1, keepdim=True) & (lam > 0)
        level = _blocks(x, held)
        x -= level
        dec = x.square().sum(1, keepdim=True)
        done = (~inward & (dec <= n * (10 * floor).square())).view(-1)
        out[left[done]] = level[done]
        if bool(done.all()):
            return out
        if int(done.sum()) * 4 >= done.numel():
            go = ~done
            y, u, x, held, lam, f, dec, floor, left = (t[go] for t in (y, u, x, held, lam, f, dec, floor, left))
        d = x.cumsum(1)[:, :-1].masked_fill_(held, 0.0)
        alpha = torch.ones_like(lam)
        for _ in range(40):
            new = torch.clamp(u - alpha * d, -lam, lam)
            fn = 0.5 * _primal(y, new).square().sum(1, keepdim=True)
            short = fn > f - 1e-4 * alpha * dec + 1e-15 * f
            if not bool(short.any()):
                break
            alpha = torch.where(short, 0.5 * alpha, alpha)
        u = new
    return None


def _prox64_2d(y, lam, sweeps):
    B, C, H, W = y.shape
    lam = lam.expand(C).repeat(B)
    Y, P, Q = y, torch.zeros_like(y), torch.zeros_like(y)
    for _ in range(sweeps):
        A = Y + P
        Z = _prox64(A.reshape(-1, W), lam.repeat_interleave(H).view(-1, 1))
        if Z is None:
            return None
        Z = Z.view_as(y)
        P = A - Z
        A = Z + Q
        Y = _prox64(A.transpose(2, 3).reshape(-1, H), lam.repeat_interleave(W).view(-1, 1))
        if Y is None:
            return None
        Y = Y.view(B, C, W, H).transpose(2, 3)
        Q = A - Y
    return Y


def exact(case, seed):
    y, lam, g = (t.double() for t in _inputs(case, seed))
    B, C, H, W = y.shape
    cols = case["path"] == "cols"
    if case["direction"] == "backward":
        x = _solution(case, seed)
        if cols:
            x, g = x.transpose(2, 3), g.transpose(2, 3)
        shape, n = g.shape, g.shape[-1]
        x, g = x.reshape(-1, n), g.reshape(-1, n)
        step = x[:, 1:] - x[:, :-1]
        mean = _blocks(g, step != 0)
        terms = (step.double().sign() * (mean[:, :-1] - mean[:, 1:])).sum(1)
        per = terms.view(B, C, -1)
        gl = {"scalar": per.sum().view(1), "channel": per.sum((0, 2)), "row": terms}[case["lam"]]
        gy = mean.view(shape)
        return {"grad_y": (gy.transpose(2, 3) if cols else gy).contiguous(), "grad_lam": gl}
    if case["path"] == "planes":
        x = _prox64_2d(y, lam, case["sweeps"])
    else:
        rows = y.transpose(2, 3).reshape(-1, H) if cols else y.reshape(-1, W)
        if case["lam"] == "channel":
            lam = lam.repeat(B).repeat_interleave(W if cols else H)
        x = _prox64(rows, lam.expand(len(rows)).reshape(-1, 1))
        if x is not None:
            x = x.view(B, C, W, H).transpose(2, 3) if cols else x.view_as(y)
    if x is None:
        return None
    x = x.contiguous()
    # the gradients of a whole pass have no such value: they jump wherever two levels of x meet
    return {"x": x} if case["direction"] == "infer" else {"x": x, "grad_y": None, "grad_lam": None}
