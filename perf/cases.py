"""Workloads of the fused-tile library, as a program that uses it runs them: whole early-layer networks, groups of
layers and single layers, through `harness.Session` (torch buffers around the C ABI) and the allocation-free forward
call.  A case is a network in text form plus the batch, the image, the tile grid, the grouping, the storage type and
what is called:

  op "forward"  inference with the caller's workspace; returns y
  op "static"   inference with the library's own workspace (ftp_forward_static); returns y
  op "step"     forward, back-propagation, sum of the per-stack gradients; returns y, dx and the whole gradient vector

Network text: layers separated by blanks; "c3:64-128" is a 3x3 convolution from 64 to 128 channels, "c7/2:3-64" one of
stride 2, a trailing "b" gives it a bias, "p" is the 2x2 max-pool.
"""
import math

import torch

from ftp_synth.configs import CONV, MAXPOOL, Layer
from paper_2409_09083_amd import binding as B
from paper_2409_09083_amd.harness import Session

# The early layers of the detection network of the repository's largest configurations (16 primitive layers).
_STACK16 = ("c3:3-32 p c3:32-64 p c3:64-128 c1:128-64 c3:64-128 p c3:128-256 c1:256-128 c3:128-256 p "
            "c3:256-512 c1:512-256 c3:256-512 c1:512-256")
_SMALL5 = "c3:3-16 p c3:16-32 p c3:32-64"
_SMALL12 = "c3:3-16 p c3:16-32 p c3:32-64 c3:64-128 p c1:128-64 c3:64-128 p c1:128-64 c3:64-128"
_STEM = "c7/2:3-64 p c3:64-64 c3/2:64-128 c1:128-64 c5:64-128 p c3/2:128-256 p c3:256-256"


def _case(name, net, batch, h, w, grid, groups, dtype="f32", op="step", slope=0.1):
    c = {"net": net, "batch": batch, "h": h, "w": w, "grid_n": grid[0], "grid_m": grid[1],
         "groups": ",".join(str(g) for g in groups), "dtype": dtype, "op": op, "slope": slope}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a few kernels of a few microseconds each, bound by launches.
        _case("tiny_step", "c3:3-8 c3:8-16", 1, 32, 32, (2, 2), (2,)),
        # One camera image through the fixed workspace: serving latency.
        _case("image_static_f32", _SMALL5, 1, 416, 416, (3, 3), (5,), op="static"),
        # Training on one image at a time, the edge-device setting.
        _case("image_step_f32", _SMALL5, 1, 416, 416, (3, 3), (5,)),
        # A small network at an ordinary batch.
        _case("small_net_step_f32", _SMALL12, 8, 608, 608, (4, 4), (7, 12)),
        # The headline training step: 16 layers, 64 images, 6 x 6 tiles.
        _case("net_step_f32", _STACK16, 64, 608, 608, (6, 6), (4, 8, 12, 16)),
        # Batch inference with 16-bit storage, 8 x 8 tiles.
        _case("net_forward_bf16", _STACK16, 32, 608, 608, (8, 8), (4, 8, 12, 16), "bf16", op="forward"),
        # Training, 16-bit storage, the layers one at a time where they matter most: the first layer with its pool ...
        _case("stem_block_bf16", "c3:3-32 p", 32, 608, 608, (8, 8), (2,), "bf16"),
        # ... a pooled layer of the second stage ...
        _case("pool_block_bf16", "c3:32-64 p", 32, 304, 304, (8, 8), (2,), "bf16"),
        # ... and a bottleneck pair on maps that no tile divides evenly.
        _case("bottleneck_bf16", "c1:256-128 c3:128-256", 32, 76, 76, (8, 8), (2,), "bf16"),
        # A linear 3x3 pair (no activation, so its gradients have no kinks), ordinary sizes.
        _case("linear_pair_f32", "c3:64-128 c3:128-128", 16, 76, 76, (3, 3), (1, 2), slope=1.0),
        # General geometry on odd maps: large and strided filters, pools on odd maps, a bias.
        _case("odd_stem_step_f32", _STEM, 32, 607, 607, (3, 3), (3, 6, 10)),
        # Ragged everything: odd map, channel counts off the powers of two, uneven grid, biases, one image.
        _case("ragged_step_f32", "c3:24-40b c1:40-36b c3:36-72b", 1, 77, 53, (3, 5), (2, 3), slope=1.0),
    ]


def _parse(case):
    layers, c = [], None
    for t in case["net"].split():
        if t == "p":
            layers.append(Layer(MAXPOOL, 2, 2, 0, c, c, 1.0))
            continue
        head, chans = t.split(":")
        bias = chans.endswith("b")
        cin, c = (int(v) for v in chans.rstrip("b").split("-"))
        k, _, s = head[1:].partition("/")
        ly = Layer(CONV, int(k), int(s or 1), int(k) // 2, cin, c, float(case["slope"]))
        if bias:
            object.__setattr__(ly, "has_bias", 1)
        layers.append(ly)
    return layers


def _shapes(case):
    layers = _parse(case)
    out = [(layers[0].cin, case["h"], case["w"])]
    for ly in layers:
        h, w = ly.out_hw(*out[-1][1:])
        out.append((ly.cout, h, w))
    return layers, out


def _has_bias(ly):
    return bool(getattr(ly, "has_bias", 0))


def work(case):
    layers, sh = _shapes(case)
    es = 2 if case["dtype"] == "bf16" else 4
    n = case["batch"]
    passes = 3 if case["op"] == "step" else 1
    flops = params = 0
    for ly, (c, h, w) in zip(layers, sh[1:]):
        if ly.kind == CONV:
            flops += 2.0 * passes * n * h * w * ly.cout * ly.cin * ly.k * ly.k
            params += ly.cout * ly.cin * ly.k * ly.k + (ly.cout if _has_bias(ly) else 0)
    maps = n * (math.prod(sh[0]) + math.prod(sh[-1])) * es
    bytes_ = params * es + maps
    if case["op"] == "step":
        bytes_ += maps + 4 * params          # dy and dx, the gradient vector
    return {"bytes": float(bytes_), "flops": flops}


# ---- drawn cases ---------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A channel count of the sort networks have: mostly multiples of 16 or 32, sometimes only of 4."""
    v = _log(rng, lo, hi)
    step = rng.choice((4, 16, 16, 32, 32))
    return max(step, (v + step // 2) // step * step)


_LARGEST = None


def _cost(case):
    wk = work(case)
    layers, sh = _shapes(case)
    es = 2 if case["dtype"] == "bf16" else 4
    maps = case["batch"] * es * sum(math.prod(s) for s in sh)
    return wk["flops"] / (2e14 if es == 2 else 6e13) + 3 * maps / 2e12


def draw(rng):
    """One case of the ranges above: prefixes of the networks, pairs and single layers, batch 1 to 64, maps of 13 to 608
    pixels a side (odd ones too), grids from 1 x 1 to 8 x 8, both storage types, all three calls."""
    global _LARGEST
    if _LARGEST is None:
        _LARGEST = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("net", "net", "pair", "layer", "layer"))
        dtype = rng.choice(("f32", "f32", "bf16"))
        op = rng.choice(("step", "step", "step", "forward"))
        slope = rng.choice((0.1, 0.1, 1.0))
        batch = _log(rng, 1, 64)
        if kind == "net":
            net = rng.choice((_SMALL5, _SMALL12, _STACK16, _STEM)).split()
            if op == "step":
                net = net[:rng.choice((2, 3, 5, 8, len(net)) if dtype == "f32" else (2, 3))]
            h, w = _log(rng, 128, 608), _log(rng, 128, 608)
        else:
            k, s = rng.choice((("3", 1), ("3", 1), ("3", 1), ("1", 1), ("1", 1), ("3/2", 2), ("5", 1)))
            ci, co, c2 = _width(rng, 16, 512), _width(rng, 16, 512), _width(rng, 16, 256)
            bias = "b" if dtype == "f32" and rng.random() < 0.15 else ""
            net = ["c%s:%d-%d%s" % (k, ci, co, bias)]
            if kind == "pair":
                net.append(rng.choice(("p", "c1:%d-%d" % (co, c2), "c3:%d-%d" % (co, c2))))
            elif rng.random() < 0.2:
                net = [rng.choice(("c3:3-32", "c3:3-16", "c7/2:3-64", "c3/2:3-32"))]
            h, w = _log(rng, 13, 304), _log(rng, 13, 304)
        if rng.random() < 0.4:
            w = h
        case = _case(None, " ".join(net), batch, h, w, (1, 1), (1,), dtype, op, slope)
        layers, sh = _shapes(case)
        most = min(8, min(min(s[1:]) for s in sh) // 2)
        if most < 1:
            continue
        case["grid_n"] = rng.randint(1, most)
        case["grid_m"] = case["grid_n"] if rng.random() < 0.6 else rng.randint(1, most)
        g = rng.choice((1, 2, 4, len(layers)))
        ends = list(range(g, len(layers), g)) + [len(layers)]
        case["groups"] = ",".join(str(e) for e in ends)
        try:
            sizes = _sizes(case, layers)
        except B.FtpError:
            continue                          # the grid does not fit the maps
        if op == "forward" and sizes["workspace_bytes"] <= B.FTP_STATIC_WORKSPACE_BYTES and rng.random() < 0.5:
            case["op"] = "static"
        if _cost(case) <= _LARGEST and sizes["workspace_bytes"] + sizes["wgrad_partial_bytes"] < 24e9:
            return case


def _sizes(case, layers):
    plan = B.ftp_plan(layers, case["batch"], layers[0].cin, case["h"], case["w"], case["grid_n"], case["grid_m"],
                      [int(e) for e in case["groups"].split(",")], B.FTP_BF16 if case["dtype"] == "bf16" else B.FTP_F32)
    try:
        return B.ftp_plan_sizes(plan)
    finally:
        B.ftp_plan_destroy(plan)


# ---- inputs, the call ----------------------------------------------------------------------------------------------
def _inputs(case, seed):
    """x ~ U[0, 1) as an image, filters ~ N(0, 2 / (Cin K^2)), dy ~ N(0, 1); biases small.  On the GPU, from the seed."""
    layers, sh = _shapes(case)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(shape, std):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=g).to(dt)

    n = case["batch"]
    x = torch.empty((n,) + sh[0], device="cuda").uniform_(0.0, 1.0, generator=g)
    if layers[0].cin > 3:
        x = x * 2 - 0.5                       # an activation map rather than an image: both signs
    weights = [normal((ly.cout, ly.cin, ly.k, ly.k), math.sqrt(2.0 / (ly.cin * ly.k * ly.k))) if ly.kind == CONV else None
               for ly in layers]
    biases = [normal((ly.cout,), 0.1) if _has_bias(ly) else None for ly in layers]
    dy = normal((n,) + sh[-1], 1.0) if case["op"] == "step" else None
    return layers, x.to(dt), weights, biases, dy


def prepare(case, seed):
    layers, x, weights, biases, dy = _inputs(case, seed)
    s = Session(layers, case["batch"], layers[0].cin, case["h"], case["w"], (case["grid_n"], case["grid_m"]),
                [int(e) for e in case["groups"].split(",")], case["dtype"])
    s.x.copy_(x)
    s.weights = weights
    if any(b is not None for b in biases):
        s.biases = biases
    if dy is not None:
        s.dy.copy_(dy)
    return {"session": s, "op": case["op"]}


def run(state):
    s = state["session"]
    if state["op"] == "forward":
        s.forward()
        return {"y": s.y}
    if state["op"] == "static":
        B.ftp_forward_static(s.plan, s.x.data_ptr(), s._wptrs(), s._bptrs(), s.y.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
        return {"y": s.y}
    s.step()
    return {"y": s.y, "dx": s.dx, "dw": s.wgrad}


# ---- what the outputs may differ by --------------------------------------------------------------------------------
def _smooth(case):
    """No pool and no kink in the activation: gradients are continuous in the forward values."""
    return float(case["slope"]) == 1.0 and "p" not in case["net"].split()


def tolerance(case):
    # Each about four times the largest difference between the default kernels and the plain direct kernels
    # (FTP_KERNELS=direct: other summation orders) over the listed and thirty drawn cases.
    bf = case["dtype"] == "bf16"
    if case["op"] != "step" or _smooth(case):
        # 32-bit sums in another order (seen: 1.9e-6, largest entry 1.2e-5); with 16-bit storage a stored value may
        # round the other way (seen: 4.4e-3, largest entry 0.028, the whole network)
        return {"rel": 2e-2, "max": 0.12} if bf else {"rel": 1e-5, "max": 1e-4}
    # A forward value within rounding of the activation's kink, or of the other candidates of its pool window, may fall
    # on the other side: a few of a gradient's entries then change by their own size (seen: 4.1e-3, largest entry 0.63).
    return {"rel": 2e-2, "max": 0.99}


def _conv64(x, w, b, stride):
    """Convolution as one product per filter tap."""
    k = w.shape[-1]
    p = k // 2
    n, _, h, wd = x.shape
    ho, wo = (h + 2 * p - k) // stride + 1, (wd + 2 * p - k) // stride + 1
    xp = torch.nn.functional.pad(x, (p, p, p, p))
    out = None
    for ky in range(k):
        for kx in range(k):
            v = xp[:, :, ky:ky + (ho - 1) * stride + 1:stride, kx:kx + (wo - 1) * stride + 1:stride]
            t = torch.matmul(w[:, :, ky, kx], v.reshape(n, v.shape[1], ho * wo))
            out = t if out is None else out + t
    if b is not None:
        out = out + b[:, None]
    return out.reshape(n, -1, ho, wo)


def exact(case, seed):
    """The same network in 64 bits.  Where activations have kinks or pools choose, a gradient has no value that rounding
    in the forward pass leaves alone (see tolerance()): only y is given."""
    layers, x, weights, biases, dy = _inputs(case, seed)
    ws = [None if w is None else w.double() for w in weights]
    bs = [None if b is None else b.double() for b in biases]
    grads = case["op"] == "step" and _smooth(case)
    params = [t for w, b in zip(ws, bs) for t in (w, b) if t is not None] if grads else []
    for t in params:
        t.requires_grad_(True)
    step = max(1, min(case["batch"], int(4e8 / (math.prod(max(_shapes(case)[1], key=math.prod)) * 8))))
    ys, dxs, total = [], [], None
    with torch.set_grad_enabled(grads):
        for at in range(0, case["batch"], step):
            v = x0 = x[at:at + step].double().requires_grad_(grads)
            for ly, w, b in zip(layers, ws, bs):
                if ly.kind == CONV:
                    v = _conv64(v, w, b, ly.stride)
                    v = torch.where(v > 0, v, v * ly.slope)
                else:
                    v = torch.nn.functional.max_pool2d(v, 2)
            ys.append(v.detach())
            if grads:
                got = torch.autograd.grad(v, [x0] + params, dy[at:at + step].double())
                dxs.append(got[0])
                total = list(got[1:]) if total is None else [s + t for s, t in zip(total, got[1:])]
    y = torch.cat(ys)
    if case["op"] != "step":
        return {"y": y}
    if not grads:
        return {"y": y, "dx": None, "dw": None}
    return {"y": y, "dx": torch.cat(dxs), "dw": torch.cat([t.reshape(-1) for t in total])}
