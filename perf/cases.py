"""The performance cases of the im2win convolution.

Each case is one call of the framework as a program makes it, on tensors that
such a program already holds on the GPU:

- op "im2win": ``transform`` into a kept window tensor, then ``conv2d`` from it
  (Alg. 2 as the paper runs it);
- op "fused": ``conv2d_fused`` straight from the input;
- op "transform": the window tensor alone (Alg. 1).

The library has one direction (forward), two dtypes (fp32, and bf16 with fp32
accumulation and fp32 output) and two window-tensor row layouts.  The listed
layers are the repository's own workloads and Table 1 layers, the same layers
in the other dtype or at batch 1, and layers whose sizes are whole multiples
of nothing.
"""
import math

import torch

import paper_2306_14320_amd as P

_FIELDS = ("n", "c", "h", "w", "k", "fh", "fw", "sh", "sw", "ph", "pw")
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
_LAYOUT = {"padded": P.IM2WIN_ROWS_PADDED, "trimmed": P.IM2WIN_ROWS_TRIMMED}


def _case(op, dtype, shape, layout="padded", name=None):
    c = dict(zip(_FIELDS, shape), op=op, dtype=dtype, layout=layout)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest workload: one 32x32 image, where launches and host calls count
        _case("im2win", "f32", (1, 3, 32, 32, 16, 3, 3, 1, 1, 0, 0), name="single_f32_im2win"),
        # one image through a mid-network layer: latency of a served request
        _case("fused", "f32", (1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1), name="one_image_f32_fused"),
        # the headline workload, the two calls of the paper's method
        _case("im2win", "f32", (32, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1), name="resnet_f32_im2win"),
        # a network's first layer: three channels, 7x7, stride 2
        _case("fused", "f32", (32, 3, 224, 224, 64, 7, 7, 2, 2, 3, 3), name="stem_f32_fused"),
        # rectangular filter, stride 2, rows trimmed to the columns that windows read
        _case("im2win", "f32", (64, 128, 28, 28, 128, 3, 5, 2, 2, 1, 2), "trimmed", "rect_f32_im2win_trimmed"),
        # the largest Table 1 layer (Conv4) at the paper's batch
        _case("im2win", "f32", (128, 64, 224, 224, 64, 7, 7, 2, 2, 0, 0), name="conv4_f32_im2win"),
        # sizes that are multiples of no tile, in fp32
        _case("fused", "f32", (6, 37, 45, 61, 75, 3, 3, 1, 1, 1, 1), name="ragged_f32_fused"),
        # a deep 14x14 layer in bf16
        _case("im2win", "bf16", (128, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1), name="deep_bf16_im2win"),
        # the headline layer in bf16
        _case("fused", "bf16", (32, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1), name="resnet_bf16_fused"),
        # the first layer in bf16
        _case("fused", "bf16", (32, 3, 224, 224, 64, 7, 7, 2, 2, 3, 3), name="stem_bf16_fused"),
        # odd sizes and stride 2 in bf16
        _case("im2win", "bf16", (5, 52, 33, 47, 90, 3, 3, 2, 2, 1, 1), name="ragged_bf16_im2win"),
        # the transformation alone: Table 1 Conv9 at the paper's batch, bound by memory
        _case("transform", "f32", (128, 64, 56, 56, 64, 3, 3, 1, 1, 0, 0), name="conv9_f32_transform"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A layer of the listed ones' ranges: batches of 1 to 128, 3 to 512 input
    and 16 to 512 output channels, 7 to 227 input rows and columns, the
    filters of the workloads and of Table 1 and 1x1, at most 100 GFLOP and
    6 GB of window tensor (under the largest listed case)."""
    while True:
        fh, fw = rng.choice([(3, 3), (3, 3), (3, 3), (1, 1), (3, 5), (5, 5), (7, 7), (11, 11)])
        c = 3 if fh == 11 or rng.random() < 0.2 else _log_int(rng, 4, 512)
        k = _log_int(rng, 16, 512)
        h = _log_int(rng, 7, 227)
        w = h if rng.random() < 0.6 else max(7, min(227, int(round(h * rng.uniform(0.6, 1.6)))))
        if rng.random() < 0.5:   # the widths that networks use
            c, k = (c if c == 3 else max(16, c // 16 * 16)), k // 16 * 16
        s = 4 if fh == 11 else rng.choice([1, 1, 2])
        half = rng.random() < 0.6
        n = _log_int(rng, 1, 128)
        case = _case(rng.choice(["im2win", "im2win", "im2win", "im2win", "fused", "fused", "fused", "fused", "transform"]),
                     rng.choice(["f32", "bf16"]),
                     (n, c, h, w, k, fh, fw, s, s, fh // 2 if half else 0, fw // 2 if half else 0),
                     rng.choice(["padded", "padded", "padded", "trimmed"]))
        ho, wo = _out(case)
        if ho < 1 or wo < 1 or _flops(case) > 100e9 or _ws_elems(case) * _elem(case) > 6e9:
            continue
        return case


def _elem(c):
    return 4 if c["dtype"] == "f32" else 2


def _out(c):
    return (c["h"] + 2 * c["ph"] - c["fh"]) // c["sh"] + 1, (c["w"] + 2 * c["pw"] - c["fw"]) // c["sw"] + 1


def _flops(c):
    ho, wo = _out(c)
    return 2 * c["n"] * c["k"] * c["c"] * ho * wo * c["fh"] * c["fw"]


def _ws_elems(c):
    ho, wo = _out(c)
    cols = (wo - 1) * c["sw"] + c["fw"] if c["layout"] == "trimmed" else c["w"] + 2 * c["pw"]
    return c["n"] * c["c"] * ho * cols * c["fh"]


def _tensors(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    xs, wsz = (c["n"], c["c"], c["h"], c["w"]), (c["k"], c["c"], c["fh"], c["fw"])
    if c["c"] == 3:   # normalised images
        x = torch.randn(xs, generator=g, device="cuda")
    else:             # activations
        x = torch.rand(xs, generator=g, device="cuda")
    w = torch.randn(wsz, generator=g, device="cuda") * math.sqrt(2.0 / (c["c"] * c["fh"] * c["fw"]))
    return x.to(_DTYPE[c["dtype"]]), w.to(_DTYPE[c["dtype"]])


def prepare(case, seed):
    """Input and weights, and what a program keeps between calls: the
    descriptor, the output, the window tensor and the filter scratch."""
    x, w = _tensors(case, seed)
    d = P.desc_for(x.shape, w.shape, (case["sh"], case["sw"]), (case["ph"], case["pw"]), x.dtype,
                   _LAYOUT[case["layout"]])
    s = {"op": case["op"], "x": x, "w": w, "desc": d}
    if case["op"] != "fused":
        s["ws"] = torch.empty(P.workspace_shape(d), dtype=x.dtype, device="cuda")
    if case["op"] != "transform":
        s["y"] = torch.empty(P.y_shape(d), dtype=torch.float32, device="cuda")
        s["scratch"] = P.filter_scratch(d, "cuda")
    return s


def run(s):
    if s["op"] == "fused":
        return P.conv2d_fused(s["x"], s["w"], s["desc"], y=s["y"], scratch=s["scratch"])
    ws = P.transform(s["x"], s["desc"], ws=s["ws"])
    if s["op"] == "transform":
        return ws
    return P.conv2d(ws, s["w"], s["desc"], y=s["y"], scratch=s["scratch"])


def work(case):
    """The input and the weights read once, the output written once; an
    im2win pass also writes its window tensor and reads it back."""
    ho, wo = _out(case)
    e = _elem(case)
    x, w = e * case["n"] * case["c"] * case["h"] * case["w"], e * case["k"] * case["c"] * case["fh"] * case["fw"]
    y, ws = 4 * case["n"] * case["k"] * ho * wo, e * _ws_elems(case)
    if case["op"] == "transform":
        return {"bytes": x + ws, "flops": 0}
    return {"bytes": x + w + y + (2 * ws if case["op"] == "im2win" else 0), "flops": _flops(case)}


def tolerance(case):
    """The transformation copies.  Products and sums are fp32 for both dtypes
    (bf16 products are exact in fp32); the listed and drawn layers measure up
    to 1.1e-6 against 64 bits."""
    return "exact" if case["op"] == "transform" else {"rel": 5e-6}


def exact(case, seed):
    """The convolution in 64 bits: the im2col matrix of a few images at a time
    times the filter matrix."""
    if case["op"] == "transform":
        return None
    x, w = _tensors(case, seed)
    ho, wo = _out(case)
    wm = w.double().reshape(case["k"], -1)
    y = torch.empty((case["n"], case["k"], ho * wo), dtype=torch.float64, device="cuda")
    step = max(1, int(4e9 // (8 * wm.shape[1] * ho * wo)))
    for i in range(0, case["n"], step):
        cols = torch.nn.functional.unfold(x[i:i + step].double(), (case["fh"], case["fw"]),
                                          padding=(case["ph"], case["pw"]), stride=(case["sh"], case["sw"]))
        for j in range(cols.shape[0]):
            torch.mm(wm, cols[j], out=y[i + j])
    return y.view(case["n"], case["k"], ho, wo)
