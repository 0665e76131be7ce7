"""Timed cases of the convolution library: what a program does with it, through its public entry points.

A case is one or more convolution layers and the operations run on each: Forward alone (inference) or
Forward, BackwardData and BackwardFilter (a training step).  The program holds its tensors, a workspace
of the limit that it planned for, and the plans that `ucd_plan` made for it on its own buffers; a pass
is the `ucd_conv_*` calls.  Sizes come from the layer tables in `paper_1804_04806_amd/synth.py`.
"""
import math

import torch
import torch.nn.functional as F

from paper_1804_04806_amd import synth, ucd

KIB, MIB = 1 << 10, 1 << 20


def _one(name, ops, dtype, ws, n, c, h, w, k, r, s, stride, pad_h, pad_w):
    return {"name": name, "net": "", "ops": ops, "dtype": dtype, "ws_bytes": ws, "N": n, "C": c, "H": h, "W": w,
            "K": k, "R": r, "S": s, "stride": stride, "pad_h": pad_h, "pad_w": pad_w}


def listed():
    return [
        # the smallest call: a layer whose kernels take microseconds, no room for workspace
        _one("small train", "train", "f32", 64 * KIB, 8, 16, 16, 16, 32, 3, 3, 1, 1, 1),
        # one image through a deep 3x3 layer: latency of a serving call
        _one("one image 3x3", "fwd", "f32", 64 * MIB, 1, 256, 14, 14, 256, 3, 3, 1, 1, 1),
        # the library's headline workload: a training step of the AlexNet-shaped stack at batch 256
        {"name": "alexnet step", "net": "alexnet", "ops": "train", "dtype": "f32", "ws_bytes": 64 * MIB, "N": 256},
        # a ResNet's first layer: 3 input channels, 7x7 filter, stride 2
        _one("stem 7x7/2 train", "train", "f32", 64 * MIB, 128, 3, 224, 224, 64, 7, 7, 2, 3, 3),
        # the layer that residual networks repeat most
        _one("3x3 256ch 14x14 train", "train", "f32", 64 * MIB, 256, 256, 14, 14, 256, 3, 3, 1, 1, 1),
        # entry of a residual stage: strided 3x3
        _one("3x3/2 64-128 train", "train", "f32", 64 * MIB, 128, 64, 56, 56, 128, 3, 3, 2, 1, 1),
        # bottleneck expansion: 1x1, four times as many channels out as in
        _one("1x1 128-512 28x28 train", "train", "f32", 64 * MIB, 128, 128, 28, 28, 512, 1, 1, 1, 0, 0),
        # densely connected block, 8 MiB limit
        _one("1x1 352-128 32x32 train", "train", "f32", 8 * MIB, 64, 352, 32, 32, 128, 1, 1, 1, 0, 0),
        # odd and ragged in every extent, a filter that is not square
        _one("ragged 3x5 train", "train", "f32", 8 * MIB, 37, 51, 45, 29, 77, 3, 5, 1, 1, 2),
        # bf16 tensors: the AlexNet-shaped stack's largest 3x3 layer
        _one("bf16 3x3 384ch train", "train", "bf16", 64 * MIB, 256, 384, 13, 13, 384, 3, 3, 1, 1, 1),
        # bf16 bottleneck reduction
        _one("bf16 1x1 1024-256 train", "train", "bf16", 64 * MIB, 256, 1024, 14, 14, 256, 1, 1, 1, 0, 0),
        # bf16 inference at a serving batch
        _one("bf16 3x3 128ch fwd", "fwd", "bf16", 64 * MIB, 32, 128, 28, 28, 128, 3, 3, 1, 1, 1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# limits of a drawn case: below the stack's step (0.55 Tflop and 0.3 GB per operation of its larger layers),
# also where a strided layer's gradient runs at a tenth of the best rate
_MAX_FLOPS, _MAX_ELEMENTS = 1.0e11, 3.0e7


def draw(rng):
    """Any layer of the kinds above: filters 1x1 to 11x11, strides 1 to 4, 3 to 1024 channels, images of 7 to
    227 pixels, 1 to 256 of them; now and then odd filters; fp32 twice as often as bf16."""
    while True:
        r = rng.choice([1, 1, 3, 3, 3, 5, 7, 11])
        s = r if r == 1 or rng.random() < 0.8 else rng.choice([1, 3, 5, 7])
        stride = {1: rng.choice([1, 1, 1, 2]), 3: rng.choice([1, 1, 1, 2]), 5: rng.choice([1, 1, 2]),
                  7: rng.choice([1, 2, 2]), 11: rng.choice([1, 4, 4])}[r]
        same = rng.random() < 0.8
        c = 3 if r >= 7 and rng.random() < 0.6 else _log(rng, 8, 1024)
        h = _log(rng, 7, 227)
        w = h if rng.random() < 0.6 else _log(rng, 7, 227)
        pad_h, pad_w = (r // 2, s // 2) if same else (0, 0)
        case = _one("", rng.choice(["train", "train", "train", "fwd"]), rng.choice(["f32", "f32", "bf16"]),
                    rng.choice([64 * KIB, 8 * MIB, 64 * MIB, 64 * MIB]), _log(rng, 1, 256), c, h, w,
                    _log(rng, 16, 1024), r, s, stride, pad_h, pad_w)
        del case["name"]
        if h + 2 * pad_h < r or w + 2 * pad_w < s:
            continue
        lay = _layers(case)[0]
        if lay.flops <= _MAX_FLOPS and max(_elements(lay)) <= _MAX_ELEMENTS:
            return case


class _Layer:
    def __init__(self, n, c, h, w, k, r, s, stride, pad_h, pad_w):
        self.x_shape, self.w_shape = (n, c, h, w), (k, c, r, s)
        self.stride, self.pad = stride, (pad_h, pad_w)
        self.y_shape = (n, k, (h + 2 * pad_h - r) // stride + 1, (w + 2 * pad_w - s) // stride + 1)
        self.flops = 2 * math.prod(self.y_shape) * c * r * s

    def desc(self, dtype):
        (n, c, h, w), (k, _, r, s) = self.x_shape, self.w_shape
        return ucd.layer(N=n, C=c, H=h, W=w, K=k, R=r, S=s, stride_h=self.stride, stride_w=self.stride,
                         pad_h=self.pad[0], pad_w=self.pad[1], dtype=1 if dtype == "bf16" else 0)


def _layers(case):
    if case["net"]:
        return [_Layer(s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.stride, s.pad, s.pad)
                for s in getattr(synth, "config_" + case["net"])(case["N"])]
    return [_Layer(*(case[f] for f in ("N", "C", "H", "W", "K", "R", "S", "stride", "pad_h", "pad_w")))]


def _elements(lay):
    return [math.prod(t) for t in (lay.x_shape, lay.w_shape, lay.y_shape)]


def _inputs(case, seed):
    """x, w, dy of every layer: normalised pixels for a first layer and activations behind a ReLU for the others,
    He-initialised filters, zero-mean gradients."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    got = []
    for lay in _layers(case):
        def normal(shape, std=1.0):
            return torch.randn(shape, device="cuda", generator=gen).mul_(std)
        x = normal(lay.x_shape)
        if lay.x_shape[1] != 3:
            x.relu_()
        w = normal(lay.w_shape, math.sqrt(2.0 / math.prod(lay.w_shape[1:])))
        got.append((x.to(dtype), w.to(dtype), normal(lay.y_shape, 0.1).to(dtype)))
    return got


def prepare(case, seed):
    train = case["ops"] == "train"
    ws = torch.empty(case["ws_bytes"], dtype=torch.uint8, device="cuda")
    limit = case["ws_bytes"]
    layers = []
    for lay, (x, w, dy) in zip(_layers(case), _inputs(case, seed)):
        desc = lay.desc(case["dtype"])
        one = {"x": x, "w": w, "dy": dy, "y": torch.empty_like(dy)}
        one["fwd"] = ucd.ucd_plan(desc, ucd.FWD, limit, ucd.POLICY_POW2, x, w, one["y"], ws)
        if train:
            one["dx"] = torch.empty_like(x)
            one["dw"] = torch.empty(lay.w_shape, dtype=torch.float32, device="cuda")
            one["bwd_data"] = ucd.ucd_plan(desc, ucd.BWD_DATA, limit, ucd.POLICY_POW2, one["dx"], w, dy, ws)
            one["bwd_filter"] = ucd.ucd_plan(desc, ucd.BWD_FILTER, limit, ucd.POLICY_POW2, x, one["dw"], dy, ws)
        layers.append(one)
    return {"train": train, "layers": layers, "ws": ws}


def run(state):
    ws, out = state["ws"], []
    for one in state["layers"]:
        ucd.ucd_conv_fwd(one["fwd"], one["x"], one["w"], one["y"], ws)
        out.append({"y": one["y"]})
    if state["train"]:
        for one, got in zip(reversed(state["layers"]), reversed(out)):
            ucd.ucd_conv_bwd_filter(one["bwd_filter"], one["x"], one["dy"], one["dw"], 0.0, ws)
            ucd.ucd_conv_bwd_data(one["bwd_data"], one["dy"], one["w"], one["dx"], ws)
            got["dx"], got["dw"] = one["dx"], one["dw"]
    return out


def work(case):
    """Direct-convolution flops; each operand of each operation read once, each result written once."""
    e = 2 if case["dtype"] == "bf16" else 4
    nbytes = flops = 0
    for lay in _layers(case):
        x, w, y = _elements(lay)
        ops = 3 if case["ops"] == "train" else 1
        flops += ops * lay.flops
        nbytes += ops * e * (x + y) + e * w
        if ops == 3:
            nbytes += (e + 4) * w  # the filter again for BackwardData; dw is fp32 for both types
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["dtype"] == "bf16":
        # outputs rounded to 8 bits (2.3e-3), and where Winograd runs its transforms are too (4.3e-3)
        return {"rel": 1.5e-2}
    # 32-bit sums: 2e-7 to 6e-7 measured; the Winograd algorithms that the planner may choose for square
    # 3x3 and 5x5 filters reach 4e-6
    winograd = any(lay.w_shape[2:] in ((3, 3), (5, 5), (7, 7), (11, 11)) for lay in _layers(case))
    return {"rel": 1.6e-5 if winograd else 4e-6}


def exact(case, seed):
    out = []
    for lay, (x, w, dy) in zip(_layers(case), _inputs(case, seed)):
        out.append(_exact_layer(lay, x.double(), w.double(), dy.double(), case["ops"] == "train"))
    return out


def _exact_layer(lay, x, w, dy, train):
    n, k, p, q = lay.y_shape
    geom = {"kernel_size": lay.w_shape[2:], "padding": lay.pad, "stride": lay.stride}
    w2 = w.reshape(k, -1)
    got = {"y": torch.empty_like(dy)}
    if train:
        got["dx"], got["dw"] = torch.empty_like(x), torch.zeros_like(w2)
    step = max(1, int(6e7) // (w2.shape[1] * p * q))
    for o in range(0, n, step):
        part = slice(o, min(n, o + step))
        m = part.stop - part.start
        cols = F.unfold(x[part], **geom).transpose(0, 1).reshape(w2.shape[1], m * p * q)
        got["y"][part] = (w2 @ cols).reshape(k, m, p, q).transpose(0, 1)
        if train:
            g = dy[part].transpose(0, 1).reshape(k, m * p * q)
            got["dw"] += g @ cols.t()
            back = (w2.t().contiguous() @ g).reshape(w2.shape[1], m, p * q).transpose(0, 1).contiguous()
            got["dx"][part] = F.fold(back, lay.x_shape[2:], **geom)
    if train:
        got["dw"] = got["dw"].reshape(lay.w_shape)
    return got
