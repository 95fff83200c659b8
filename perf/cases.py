"""The work whose speed matters: pruned convolution layers and small networks of them, as a program that serves
them calls the library (handles made once, output buffers kept, one forward call per layer and pass).

A case is one layer (`kind` "layer") or a chain of layers with bias, ReLU and pooling (`kind` "vgg" or "lenet").
Layer shapes are those of this repository's own workloads: the single small layer, the LeNet-5-style pair, VGG-16
for 32-pixel images, the 256 -> 256 layer on 14 x 14 maps over its range of sparsities, VGG-16's layers on
224-pixel images, the 1 x 1 bottleneck layers of ResNet and DenseNet and the 1-D text model.
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2011_06295_amd import binding as B

VGG_WIDTHS = ((64, 64), (128, 128), (256, 256, 256), (512, 512, 512), (512, 512, 512))


def layer(name, dtype, n, c, k, h, w, r=3, s=3, stride=1, pad=1, sparsity=90.0, rows="unified", coded=False):
    """rows: "unified" (the same count of kept weights in every output channel) or "ragged" (counts spread around it).
    coded: the weights are given as 4-bit numbers of 16 centroids."""
    case = dict(kind="layer", dtype=dtype, n=n, c=c, k=k, h=h, w=w, r=r, s=s, stride=stride, pad=pad,
                sparsity=sparsity, rows=rows, coded=coded)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: one image through one small layer, where the launch is most of the time
        layer("single_f32_b1", "f32", 1, 16, 32, 16, 16, rows="ragged"),
        # a small network: two 5 x 5 layers with pooling and ReLU between them
        dict(kind="lenet", dtype="f32", n=64, name="lenet5_f32_b64"),
        # a whole classifier pass in both storage types: 13 layers, 80 to 95 % sparse, maps from 32 x 32 down to 2 x 2
        dict(kind="vgg", dtype="f32", n=128, name="vgg32_f32_b128"),
        dict(kind="vgg", dtype="f16", n=256, name="vgg32_f16_b256"),
        # one middle-of-the-network layer over the range of sparsities that pruning reaches
        layer("map14_f32_s70", "f32", 256, 256, 256, 14, 14, sparsity=70.0),
        layer("map14_f32_s90_ragged", "f32", 256, 256, 256, 14, 14, sparsity=90.0, rows="ragged"),
        layer("map14_f32_s99", "f32", 256, 256, 256, 14, 14, sparsity=99.0),
        # layers of a network for 224-pixel images: the largest call, and a deep layer in binary16
        layer("map112_f32_s90", "f32", 128, 64, 128, 112, 112),
        layer("map28_f16_s90", "f16", 128, 256, 512, 28, 28),
        # 1 x 1 bottlenecks: wide output on large maps, and a long reduction on odd maps with 4-bit weights
        layer("point56_f16_s90", "f16", 128, 64, 256, 56, 56, 1, 1, 1, 0),
        layer("point7_coded_s91", "f32", 128, 1776, 192, 7, 7, 1, 1, 1, 0, sparsity=91.0, coded=True),
        # a text model: 1-D convolution over 64 words of 300 dimensions
        layer("text_f32_s83", "f32", 128, 300, 100, 1, 64, 1, 3, 1, 0, sparsity=83.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; layers cost at most what the largest listed one costs (stored multiply-adds
    and bytes are both capped well below it)."""
    while True:
        dtype = rng.choice(("f32", "f16"))
        what = rng.choice(("map", "map", "map", "map", "point", "point", "text", "first", "strided", "vgg"))
        if what == "vgg":
            return dict(kind="vgg", dtype=dtype, n=_log_int(rng, 1, 200))
        n = _log_int(rng, 1, 256)
        sparsity = rng.choice((50.0, 70.0, 80.0, 87.5, 90.0, 91.0, 93.0, 95.0, 99.0))
        rows = rng.choice(("unified", "unified", "ragged"))
        coded = rng.random() < 0.15
        c, k = _log_int(rng, 16, 512), _log_int(rng, 16, 512)
        if what == "map":          # 3 x 3 and now and then 5 x 5, maps from 2 x 2 to 112 x 112
            r = rng.choice((3, 3, 3, 5))
            h = _log_int(rng, 2 if r == 3 else 6, 112)
            case = layer("", dtype, n, c, k, h, h, r, r, 1, r // 2, sparsity, rows, coded)
        elif what == "point":      # 1 x 1
            h = _log_int(rng, 7, 56)
            case = layer("", dtype, n, _log_int(rng, 64, 1776), k, h, h, 1, 1, 1, 0, sparsity, rows, coded)
        elif what == "text":       # 1-D
            case = layer("", dtype, n, 300, _log_int(rng, 50, 200), 1, _log_int(rng, 24, 128), 1, rng.choice((2, 3)), 1, 0,
                         sparsity, rows, coded)
        elif what == "first":      # a network's first layer: few input channels, large maps
            h = _log_int(rng, 28, 224)
            case = layer("", dtype, n, rng.choice((1, 3)), k, h, h, 3, 3, 1, 1, rng.choice((50.0, 70.0, 80.0)), rows, coded)
        else:                      # stride 2
            h = _log_int(rng, 8, 112)
            case = layer("", dtype, n, c, k, h, h, 3, 3, 2, 1, sparsity, rows, coded)
        cost = work(case)
        if cost["flops"] <= 2e10 and cost["bytes"] <= 1e9:
            return case


# ---------------------------------------------------------------- shapes and work

def _convs(case):
    """The layers of a case, each (c, k, h, w, r, s, stride, pad, sparsity, pool after it)."""
    if case["kind"] == "layer":
        return [(case["c"], case["k"], case["h"], case["w"], case["r"], case["s"], case["stride"], case["pad"], case["sparsity"], False)]
    if case["kind"] == "lenet":
        return [(1, 20, 28, 28, 5, 5, 1, 0, 90.0, True), (20, 50, 12, 12, 5, 5, 1, 0, 90.0, False)]
    out, c, h = [], 3, 32
    for group in VGG_WIDTHS:
        for i, k in enumerate(group):
            out.append((c, k, h, h, 3, 3, 1, 1, 80.0 + 1.25 * len(out), i == len(group) - 1))
            c = k
        h //= 2
    return out


def _kept(length, sparsity):
    return max(1, int(length * (100.0 - sparsity) / 100.0 + 0.5))


def work(case):
    """Multiply-adds of the stored weights; the input, every stored weight with its position, and the output once.
    (Between the layers of a chain the activations need not leave the chip.)"""
    b = 2 if case["dtype"] == "f16" else 4
    flops = nbytes = 0
    convs = _convs(case)
    for i, (c, k, h, w, r, s, stride, pad, sparsity, pool) in enumerate(convs):
        e, f = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1
        nnz = k * _kept(c * r * s, sparsity)
        flops += 2 * nnz * e * f * case["n"]
        nbytes += nnz * (b + 4)
        if i == 0:
            nbytes += case["n"] * c * h * w * b
        if i == len(convs) - 1:
            nbytes += case["n"] * k * e * f * b // (4 if pool else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the largest error seen against the same path in 64 bits.  fp32: sums of up to some thousand terms in
    another order (4.6e-7 over a layer's output, 3.1e-7 after the chain).  binary16: one rounding of each output
    (2.1e-4), and in a chain of 13 layers the roundings of all of them (5.6e-4)."""
    if case["dtype"] == "f16":
        return {"rel": 2.5e-3, "max": 1e-2} if case["kind"] == "vgg" else {"rel": 8e-4, "max": 2e-3}
    return {"rel": 2e-6, "max": 1.2e-5}


# ---------------------------------------------------------------- what a program has in hand

def _mask(rng, k, length, sparsity, rows):
    """Kept weights [k][length]: the given count in every row, or counts spread around it."""
    want = _kept(length, sparsity)
    order = rng.random((k, length), dtype=np.float32)
    if rows == "unified":
        cut = np.partition(order, want - 1, axis=1)[:, want - 1:want]
        return (order <= cut).astype(np.uint8)
    density = np.clip(2.0 * want / length * rng.beta(2.0, 2.0, k), 0.0, 1.0)
    return (order < density[:, None].astype(np.float32)).astype(np.uint8)


def _handle(case, rng, conv):
    c, k, _, _, r, s, _, _, sparsity, _ = conv
    mask = _mask(rng, k, c * r * s, sparsity, case.get("rows", "unified")).reshape(k, c, r, s)
    std = math.sqrt(2.0 / _kept(c * r * s, sparsity))
    if case.get("coded"):
        centroids = np.sort(rng.standard_normal(16)).astype(np.float32) * np.float32(std)
        return B.SparseConv.from_codebook(rng.integers(0, 16, mask.shape, dtype=np.uint8), centroids, mask, dtype=case["dtype"])
    weights = rng.standard_normal(mask.shape, dtype=np.float32) * np.float32(std)
    return B.SparseConv(weights, mask, dtype=case["dtype"])


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    convs = _convs(case)
    dtype = torch.float16 if case["dtype"] == "f16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    c, _, h, w = convs[0][:4]
    x = torch.randn((case["n"], c, h, w), generator=gen, device="cuda", dtype=torch.float32).to(dtype)
    steps = []
    for i, conv in enumerate(convs):
        _, k, h, w, r, s, stride, pad, _, pool = conv
        handle = _handle(case, rng, conv)
        e, f = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1
        if case["kind"] != "layer":   # bias, activation and pooling belong to the network
            bias = 0.05 * rng.standard_normal(k).astype(np.float32)
            relu = case["kind"] == "vgg" or i == 0
            if pool:                  # in the layer's store step where the library can plan it, else after it
                handle.set_epilogue(bias, relu=relu, maxpool=True)
                try:
                    handle.get_launch(case["n"], h, w, stride, pad)
                    e, f, pool = e // 2, f // 2, False
                except B.SparseConvError:
                    handle.set_epilogue(bias, relu=relu)
            else:
                handle.set_epilogue(bias, relu=relu)
        out = torch.empty((case["n"], k, e, f), device="cuda", dtype=dtype)
        steps.append((handle, stride, pad, out, pool))
    return {"x": x, "steps": steps}


def run(state):
    y = state["x"]
    for handle, stride, pad, out, pool in state["steps"]:
        y = handle.forward(y, stride, pad, out=out)
        if pool:
            y = F.max_pool2d(y, 2)
    return y
