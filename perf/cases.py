"""The work whose speed is watched: forward passes of the CNN graphs this repository plans and runs, as a serving program makes them.

A case names a graph family of `workloads.cnn_graphs` and its sizes, the type it computes in, the link level, how the caller holds
its input and output, and the entry point of the pass.  `prepare` is what such a program does once per model (graph, plan, packed
weights, device buffers), `run` is one forward pass on the input that lies in device memory."""
from __future__ import annotations

import functools
import math

import torch
import torch.nn.functional as F

from paper_2302_00282_amd import xenos as X
from workloads import cnn_graphs as wg

#: How the caller holds the graph's input and output: (dtype, layout).
FORMATS = {"f32_nchw": (X.XENOS_F32, X.XENOS_NCHW), "bf16_nhwc": (X.XENOS_BF16, X.XENOS_NHWC)}
COMPUTE = {"f32": X.XENOS_F32, "bf16": X.XENOS_BF16}


def _case(family, batch, compute, *, hw=224, width=1.0, hidden=0, link=3, io="f32_nchw", entry="run"):
    return dict(family=family, batch=batch, hw=hw, width=width, hidden=hidden, compute=compute, link=link, io=io, entry=entry)


def listed():
    return [
        # one Conv3x3 + BN + ReLU + MaxPool chain on a 32x32 image: the smallest graph anyone runs, nothing but launches
        dict(_case("single_chain", 1, "f32", hw=32, link=2), name="single_chain_b1_f32"),
        # feed-forward block of a small transformer on 128 tokens, 512 -> 2048 -> 512 with its shortcut
        dict(_case("matmul", 128, "bf16", width=512, hidden=2048, io="bf16_nhwc"), name="matmul_128x512_bf16"),
        # one camera image through each of the mobile networks: the real-time use, every chain short and dependent on the last
        dict(_case("mobilenet", 1, "bf16"), name="mobilenet_b1_bf16"),
        dict(_case("mobilenet", 1, "f32"), name="mobilenet_b1_f32"),
        dict(_case("squeezenet", 1, "bf16", entry="graph"), name="squeezenet_b1_bf16_graph"),
        dict(_case("resnet18", 1, "bf16"), name="resnet18_b1_bf16"),
        # a part-filled server batch of odd-sized crops, held as a bf16 NHWC tensor by the caller, on a thinner network
        dict(_case("mobilenet", 7, "bf16", hw=193, width=0.75, io="bf16_nhwc"), name="mobilenet_b7_193_bf16"),
        # full server batches
        dict(_case("squeezenet", 32, "f32"), name="squeezenet_b32_f32"),
        dict(_case("squeezenet", 32, "bf16"), name="squeezenet_b32_bf16"),
        dict(_case("shufflenet", 32, "bf16"), name="shufflenet_b32_bf16"),
        dict(_case("resnet18", 32, "bf16"), name="resnet18_b32_bf16"),
        # the largest: a dense 3x3 stack and three wide fully connected layers
        dict(_case("vgg16", 32, "bf16"), name="vgg16_b32_bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any of the families at batch 1 .. 32, image sides 64 .. 256 (odd ones too), the usual width multipliers, both compute types."""
    family = rng.choice(["single_chain", "matmul", "mobilenet", "mobilenet", "squeezenet", "shufflenet", "resnet18", "vgg16"])
    compute = rng.choice(["bf16", "bf16", "f32"])
    link = rng.choice([3, 3, 3, 2])
    entry = rng.choice(["run", "run", "graph"])
    if family == "matmul":
        width = 8 * rng.randint(12, 128)
        return _case(family, _log(rng, 1, 1024), compute, width=width, hidden=4 * width, link=link, entry=entry,
                     io="bf16_nhwc" if compute == "bf16" else "f32_nchw")
    case = _case(family, _log(rng, 1, 32), compute, hw=rng.randint(64, 256), link=link, entry=entry,
                 io=rng.choice(["f32_nchw", "f32_nchw", "bf16_nhwc"]) if compute == "bf16" else "f32_nchw")
    if family in ("mobilenet", "resnet18"):
        case["width"] = rng.choice([0.25, 0.5, 0.75, 1.0])
    elif family == "vgg16":
        case["width"] = rng.choice([0.25, 0.5, 1.0])
        case["hw"] = min(case["hw"], 224)                     # (the first fully connected layer grows with the image)
    most = _price(dict(listed()[-1]))
    while case["batch"] > 1 and _price(case) > most:
        case["batch"] //= 2
    return case


def _price(case):
    return work(case)["flops"] * (16 if case["compute"] == "f32" else 1)       # (the matrix rates of the two types)


def _graph(case):
    """The graph with zeros for parameters: shapes only."""
    f, b, hw, w = case["family"], case["batch"], case["hw"], case["width"]
    if f == "matmul":
        return wg.matmul_chain(rows=b, widths=(w, case["hidden"], w), draw=False)
    if f == "single_chain":
        return wg.single_chain(batch=b, hw=hw, draw=False)
    if f == "mobilenet":
        return wg.mobilenet_v1(batch=b, hw=hw, width=w, draw=False)
    if f == "resnet18":
        return wg.resnet18(batch=b, hw=hw, width=w, draw=False)
    if f == "vgg16":
        return wg.vgg16(batch=b, hw=hw, width=w, fc_dim=int(4096 * w), draw=False)
    if f == "squeezenet":
        return wg.squeezenet11(batch=b, hw=hw, draw=False)
    return wg.shufflenet_v2(batch=b, hw=hw, draw=False)


class Model:
    """A planned graph with its weights and buffers on the GPU."""

    def __init__(self, graph, case, x):
        fmt = FORMATS[case["io"]]
        self.session = X.Session(graph, link=case["link"], split=1, compute=COMPUTE[case["compute"]], in_dtype=fmt[0], in_layout=fmt[1],
                                 out_dtype=fmt[0], out_layout=fmt[1])
        s = self.session
        s.x.copy_(x.permute(0, 2, 3, 1) if fmt[1] == X.XENOS_NHWC else x)
        self.forward = s.run_graph if case["entry"] == "graph" else s.run

    def __del__(self):
        if hasattr(self, "session"):
            self.session.close()


def _drawn(case, seed):
    """The graph with its parameters (NumPy arrays on the host) and the input on the GPU, by the recipe of `workloads.cnn_graphs`:
    He-normal weights, BN statistics around one, input U[-1, 1], drawn on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, std):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std)

    def uniform(shape, lo, hi):
        return torch.rand(shape, generator=gen, device="cuda").mul_(hi - lo).add_(lo)

    graph = _graph(case)
    for op in graph.ops:
        for key, zeros in op.params.items():
            if key == "weight":
                value = normal(zeros.shape, math.sqrt(2.0 / math.prod(zeros.shape[1:])))
            elif key in ("gamma", "var"):
                value = uniform(zeros.shape, 0.5, 1.5)
            else:
                value = normal(zeros.shape, 0.1)
            op.params[key] = value.cpu().numpy()
    return graph, uniform(graph.input_shape, -1.0, 1.0)


def prepare(case, seed):
    """The plan of the drawn graph, bound to its device memory."""
    graph, x = _drawn(case, seed)
    return Model(graph, case, x)


def run(state):
    state.forward()
    return state.session.y


@functools.lru_cache(maxsize=256)
def _work(items):
    case = dict(items)
    g = _graph(case)
    shapes = g.shapes()
    flops = 0
    for op, out in zip(g.ops, shapes[1:]):
        if op.kind in ("conv", "fc", "matmul"):
            flops += 2 * math.prod(out) * math.prod(op.params["weight"].shape[1:])
    esz = 2 if case["compute"] == "bf16" else 4
    io = 2 if case["io"] == "bf16_nhwc" else 4
    weights = sum(p.size * (esz if k == "weight" else 4) for op in g.ops for k, p in op.params.items())
    return weights + io * (math.prod(g.input_shape) + math.prod(shapes[g.output])), flops


def work(case):
    """Input, every parameter and output once; the multiply-adds of the convolutions and matrix products."""
    nbytes, flops = _work(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the logits of whole networks differ by when the same pass is planned at another link level, which sums in another
    order and rounds at other places: up to 3.7e-3 (largest value 1.5e-2) with bf16 tensors between the chains, 1.1e-6 (4.6e-6) in fp32."""
    if case["compute"] == "f32":
        return {"rel": 5e-6, "max": 2e-5}
    return {"rel": 1.5e-2, "max": 6e-2}


def _plain(op, ins):
    """One operator of the graph in torch, in the type of its inputs."""
    a, x = op.attrs, ins[0]
    p = {k: torch.from_numpy(v).to(x.device, x.dtype) for k, v in op.params.items()}
    per_channel = lambda k: p[k].view(1, -1, 1, 1)
    if op.kind == "conv":
        return F.conv2d(x, p["weight"], p.get("bias"), stride=a["stride"], padding=a["pad"], groups=a["groups"])
    if op.kind in ("fc", "matmul"):
        return F.linear(x.flatten(1), p["weight"].flatten(1), p.get("bias"))[:, :, None, None]
    if op.kind == "bias":
        return x + per_channel("bias")
    if op.kind == "bn":
        return (x - per_channel("mean")) / torch.sqrt(per_channel("var") + a["eps"]) * per_channel("gamma") + per_channel("beta")
    if op.kind == "relu":
        return x.clamp_min(0)
    if op.kind == "maxpool":
        return F.max_pool2d(x, a["k"], a["stride"], a["pad"], ceil_mode=bool(a["ceil"]))
    if op.kind == "gap":
        return x.mean((2, 3), keepdim=True)
    if op.kind == "add":
        return ins[0] + ins[1]
    if op.kind == "concat":
        return torch.cat(ins, 1)
    if op.kind == "slice":
        return x[:, a["c_begin"]:a["c_begin"] + a["out_c"]]
    assert op.kind == "shuffle", op.kind
    n, c, h, w = x.shape
    return x.view(n, a["groups"], c // a["groups"], h, w).transpose(1, 2).reshape(n, c, h, w)


def exact(case, seed):
    """The pass operator by operator in float64, a few images at a time."""
    graph, x = _drawn(case, seed)
    last = {t: i for i, op in enumerate(graph.ops) for t in op.inputs}
    parts = []
    for rows in x.split(128 if case["family"] == "matmul" else 4):
        live = {0: rows.double()}
        for i, op in enumerate(graph.ops):
            live[i + 1] = _plain(op, [live[t] for t in op.inputs])
            for t in set(op.inputs):
                if last[t] == i and t != graph.output:
                    del live[t]
        parts.append(live[graph.output])
    y = torch.cat(parts)
    return y.permute(0, 2, 3, 1).contiguous() if FORMATS[case["io"]][1] == X.XENOS_NHWC else y
