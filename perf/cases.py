"""The work that a program gives this framework: CNN inference through ``Graph``.

A program builds a graph of layers with its weights, has the routines profiled,
lets DPRS select the path (``prepare``), and then calls ``Graph.run`` on NCHW
device tensors again and again (``run``).  The cases are whole nets and the
blocks that nets are made of (stems, residual and inverted-residual blocks,
3x3 stacks, classifier heads), in the three element types, from a batch of one
image, where launches and latency count, to the largest batch in use; ``draw``
gives other sizes of the same kinds, odd and ragged ones among them.
"""

import math

import numpy as np
import torch

from paper_2110_06037_amd.graph import build_from_spec
from workloads import fuse_projection, fuse_residual, resnet18, resnet50, weight_shapes
from workloads.nets import tiny_chain

_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # the smallest whole call: a tiny fp32 classifier on one thumbnail
        {"name": "tiny_f32_bs1", "kind": "tiny", "dtype": "f32", "batch": 1},
        # single-image latency of a whole classification net
        {"name": "resnet18_bf16_bs1", "kind": "resnet18", "dtype": "bf16", "batch": 1},
        # throughput serving of a whole net: the benchmark's workload
        {"name": "resnet50_bf16_bs32", "kind": "resnet50", "dtype": "bf16", "batch": 32},
        # what images meet first: the 7x7/2 stem with its max pooling
        {"name": "stem_bf16_bs32", "kind": "stem", "dtype": "bf16", "batch": 32, "hw": 224, "c": 3, "k": 64},
        # bottleneck stages of ResNet-50 (projection block and two identity blocks):
        # large maps with few channels, bandwidth-bound
        {"name": "bottleneck56_bf16_bs32", "kind": "bottleneck", "dtype": "bf16", "batch": 32, "hw": 56, "c": 64,
         "k": 64, "stride": 1, "blocks": 3},
        # middle maps entered with stride 2, in fp16
        {"name": "bottleneck28_f16_bs32", "kind": "bottleneck", "dtype": "f16", "batch": 32, "hw": 56, "c": 256,
         "k": 128, "stride": 2, "blocks": 3},
        # small maps with many channels, at a serving batch of 8
        {"name": "bottleneck14_bf16_bs8", "kind": "bottleneck", "dtype": "bf16", "batch": 8, "hw": 28, "c": 512,
         "k": 256, "stride": 2, "blocks": 3},
        # ResNet-18 basic blocks in fp32 at a detector's odd input size
        {"name": "basic_f32_bs3_odd", "kind": "basic", "dtype": "f32", "batch": 3, "hw": 45, "c": 64, "k": 128,
         "stride": 2, "blocks": 2},
        # MobileNetV2's 28x28 inverted-residual blocks: depthwise layers, batch 8
        {"name": "inverted28_bf16_bs8", "kind": "inverted", "dtype": "bf16", "batch": 8, "hw": 56, "c": 24, "k": 32,
         "stride": 2, "blocks": 3},
        # a VGG group (two 3x3 layers and the pooling): the compute-bound end
        {"name": "vgg56_f16_bs32", "kind": "vgg", "dtype": "f16", "batch": 32, "hw": 56, "c": 128, "k": 256,
         "blocks": 3},
        # a ragged 3x3 stack: channels that are no multiple of a tile, odd map, odd batch
        {"name": "vgg_ragged_bf16_bs5", "kind": "vgg", "dtype": "bf16", "batch": 5, "hw": 37, "c": 40, "k": 72,
         "blocks": 2},
        # the classifier: global pooling and the 1000-way fully connected layer
        {"name": "head_bf16_bs32", "kind": "head", "dtype": "bf16", "batch": 32, "hw": 7, "c": 2048, "k": 1000},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["stem", "bottleneck", "bottleneck", "basic", "inverted", "vgg", "head"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    batch = _log(rng, 1, 8 if dtype == "f32" else 32)
    case = {"kind": kind, "dtype": dtype, "batch": batch}
    if kind == "stem":
        return dict(case, hw=_log(rng, 96, 256), c=rng.choice([1, 3, 3, 4]), k=8 * _log(rng, 3, 8))
    if kind == "head":
        return dict(case, hw=_log(rng, 3, 12), c=8 * _log(rng, 24, 256), k=_log(rng, 10, 1000))
    hw = _log(rng, 7, 64)
    # wider layers on smaller maps, as nets have them
    k = 8 * max(1, round(_log(rng, 256, 1024) / hw))
    case = dict(case, hw=hw, k=k, blocks=rng.randint(1, 3))
    if kind == "bottleneck":
        return dict(case, c=4 * k if hw > 14 else 2 * k, stride=rng.choice([1, 1, 2]))
    if kind == "basic":
        return dict(case, c=rng.choice([k, max(8, k // 2)]), stride=rng.choice([1, 2]))
    if kind == "inverted":
        k = max(8, k // 32 * 8)
        return dict(case, k=k, c=rng.choice([k, max(8, k // 2)]), stride=rng.choice([1, 2]))
    return dict(case, c=rng.choice([k, max(8, k // 2), max(3, k - 4)]))


def _conv(inp, k, r, stride=1, pad=None, groups=1, act="none"):
    return {"type": "conv", "in": [inp], "k": k, "r": r, "s": r, "stride": stride,
            "pad": r // 2 if pad is None else pad, "groups": groups, "act": act}


def _spec(case):
    """The net of a case in the form of ``workloads`` (structure only)."""
    kind, n, dt = case["kind"], case["batch"], case["dtype"]
    if kind == "tiny":
        return dict(tiny_chain(), batch=n)
    if kind == "resnet18":
        return fuse_residual(resnet18(n, dt))
    if kind == "resnet50":
        return fuse_projection(fuse_residual(resnet50(n, dt)))
    hw, c, k = case["hw"], case["c"], case["k"]
    layers = []

    def add(layer):
        layers.append(layer)
        return len(layers)

    x, cin = 0, c
    if kind == "stem":
        x = add(_conv(x, k, 7, 2, 3, act="relu"))
        add({"type": "maxpool", "in": [x], "k": 3, "stride": 2, "pad": 1})
    elif kind == "head":
        x = add({"type": "gap", "in": [x]})
        add({"type": "fc", "in": [x], "k": k})
    elif kind == "vgg":
        for _ in range(case["blocks"]):
            x = add(_conv(x, k, 3, act="relu"))
        add({"type": "maxpool", "in": [x], "k": 2, "stride": 2, "pad": 0})
    else:
        for b in range(case["blocks"]):
            stride, inp = case["stride"] if b == 0 else 1, x
            cout = 4 * k if kind == "bottleneck" else k
            if kind == "bottleneck":
                y = add(_conv(inp, k, 1, act="relu"))
                y = add(_conv(y, k, 3, stride, act="relu"))
                y = add(_conv(y, cout, 1))
            elif kind == "basic":
                y = add(_conv(inp, k, 3, stride, act="relu"))
                y = add(_conv(y, k, 3))
            else:
                y = add(_conv(inp, 6 * cin, 1, act="relu6"))
                y = add(_conv(y, 6 * cin, 3, stride, groups=6 * cin, act="relu6"))
                y = add(_conv(y, k, 1))
            x, same = y, stride == 1 and cin == cout
            if same or kind != "inverted":
                sc = inp if same else add(_conv(inp, cout, 1, stride, 0))
                x = add({"type": "add", "in": [y, sc], "act": "none" if kind == "inverted" else "relu"})
            cin = cout
    spec = {"name": kind, "dtype": dt, "batch": n, "in_chw": [c, hw, hw], "layers": layers}
    return fuse_projection(fuse_residual(spec))


def _draws(case, seed):
    """The input and the weights, from the seed alone: images and maps that
    follow a linear layer are centred, maps that follow a ReLU are not
    negative; He-normal weights, biases as folded batch norms leave them."""
    spec = _spec(case)
    dt = _TORCH[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = (spec["batch"], *spec["in_chw"])
    x = torch.randn(shape, generator=gen, device="cuda")
    if case["kind"] in ("bottleneck", "basic", "vgg", "head"):
        x = x.relu()
    elif case["kind"] != "inverted":
        x = x.clamp(-2.5, 2.5)

    def weight(shp):
        w = torch.randn(shp, generator=gen, device="cuda") * math.sqrt(2.0 / math.prod(shp[1:]))
        return w.to(dt)

    def bias(k):
        return torch.rand(k, generator=gen, device="cuda") * 0.2 - 0.1

    ws, bs = [], []
    for shp in weight_shapes(spec):
        if shp is None:
            ws.append(None)
            bs.append(None)
        elif len(shp) == 3:
            ws.append((weight(shp[0]), weight(shp[2])))
            bs.append((bias(shp[1]), bias(shp[1])))
        else:
            ws.append(weight(shp[0]))
            bs.append(bias(shp[1]))
    return spec, x.to(dt), ws, bs


def _host(v):
    """Host copies in the form that ``Graph`` takes (bf16 as 16-bit patterns)."""
    if v is None:
        return None
    if isinstance(v, tuple):
        return tuple(_host(e) for e in v)
    v = v.cpu()
    return v.view(torch.int16).numpy().view(np.uint16) if v.dtype == torch.bfloat16 else v.numpy()


def prepare(case, seed):
    spec, x, ws, bs = _draws(case, seed)
    # whole nets are tuned among the implicit-GEMM routines, blocks among all
    algos = ["igemm"] if case["kind"] in ("resnet18", "resnet50") else None
    g = build_from_spec(spec, {"w": [_host(w) for w in ws], "b": [_host(b) for b in bs]}, algos=algos)
    g.profile(warmup=2, reps=10)
    g.select("dprs")
    return {"g": g, "x": x, "out": g.empty_output()}


def run(state):
    return state["g"].run(state["x"], state["out"])


def work(case):
    """Input, weights and biases read once, output written once; the
    multiplications and additions of every layer."""
    spec = _spec(case)
    n, es = spec["batch"], _BYTES[case["dtype"]]
    dims = [tuple(spec["in_chw"])]
    data, flops = math.prod(spec["in_chw"]) * n, 0
    params = 0
    for layer in spec["layers"]:
        c, h, w = dims[layer["in"][0]]
        if layer["type"] in ("conv", "maxpool"):
            r = layer["r"] if layer["type"] == "conv" else layer["k"]
            h, w = ((v + 2 * layer["pad"] - r) // layer["stride"] + 1 for v in (h, w))
        if layer["type"] == "conv":
            k, per = layer["k"], c // layer["groups"] * layer["r"] * layer["s"]
            if layer.get("proj"):
                per += dims[layer["in"][1]][0]
            params += k * per * es + 4 * k
            flops += 2 * n * k * per * h * w
            c = k
        elif layer["type"] == "fc":
            params += layer["k"] * c * es + 4 * layer["k"]
            flops += 2 * n * layer["k"] * c
            c = layer["k"]
        elif layer["type"] == "maxpool":
            flops += n * c * h * w * layer["k"] ** 2
        elif layer["type"] == "gap":
            flops += n * c * h * w
            h = w = 1
        else:
            flops += n * c * h * w
        dims.append((c, h, w))
    data += n * math.prod(dims[-1])
    return {"bytes": data * es + params, "flops": flops}


def tolerance(case):
    """About four times the distance from 64 bits that was measured: one
    rounding to bf16 in the stem (1.7e-3), one or two at a head or a stack
    (2.3e-3), up to nine in a row in the blocks and whole nets (2.5e-3 to
    5.4e-3, and 2.6e-3 between two orders of ResNet-18's sums); three bits
    less in fp16 (2e-4 to 5e-4); in fp32 1.8e-6, with Winograd layers."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    rel = {"stem": 0.007, "head": 0.01, "vgg": 0.01, "inverted": 0.02}.get(case["kind"], 0.015)
    return {"rel": rel if case["dtype"] == "bf16" else rel / 8}


def _conv64(x, w, b, stride, pad, groups):
    n, c, h, wd = x.shape
    k, _, r, s = w.shape
    p, q = (h + 2 * pad - r) // stride + 1, (wd + 2 * pad - s) // stride + 1
    x = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    out = torch.zeros(n, k, p, q, dtype=x.dtype, device=x.device)
    for i in range(r):
        for j in range(s):
            t = x[:, :, i:i + (p - 1) * stride + 1:stride, j:j + (q - 1) * stride + 1:stride]
            if groups > 1:
                out += t * w[:, 0, i, j].view(1, k, 1, 1)
            else:
                rows = t.permute(0, 2, 3, 1).reshape(-1, c) @ w[:, :, i, j].t().contiguous()
                out += rows.view(n, p, q, k).permute(0, 3, 1, 2)
    return out + b.view(1, k, 1, 1)


def exact(case, seed):
    spec, x, ws, bs = _draws(case, seed)

    def wide(v):
        return v.double() if v is not None else None

    ys = [x.double()]
    for layer, w, b in zip(spec["layers"], ws, bs):
        t, y = layer["type"], ys[layer["in"][0]]
        if t == "conv" and layer.get("proj"):
            sc = ys[layer["in"][1]]
            y = _conv64(y, wide(w[0]), wide(b[0]), layer["stride"], layer["pad"], 1) + _conv64(
                sc, wide(w[1]), wide(b[1]), layer["proj"]["stride"], 0, 1)
        elif t == "conv":
            y = _conv64(y, wide(w), wide(b), layer["stride"], layer["pad"], layer["groups"])
            if len(layer["in"]) > 1:
                y = y + ys[layer["in"][1]]
        elif t == "maxpool":
            y = torch.nn.functional.max_pool2d(y, layer["k"], layer["stride"], layer["pad"])
        elif t == "gap":
            y = y.mean((2, 3), keepdim=True)
        elif t == "add":
            y = y + ys[layer["in"][1]]
        else:
            y = (y.flatten(1) @ wide(w).t() + wide(b)).view(y.shape[0], -1, 1, 1)
        act = layer.get("act", "none")
        if act != "none":
            y = y.clamp(0, 6) if act == "relu6" else y.relu()
        ys.append(y)
    y = ys[-1]
    return y.flatten(1) if y.shape[2] == y.shape[3] == 1 else y
