"""Performance cases: the blocks a user of the library has it evaluate, through the public binding.

Four families, each over a range of sizes that `draw` samples and `listed` stands for:

  matmul   products C = A B of the three layouts a Linear layer meets (nn: both row-major; nt: B stored [n][k], the layout
           of a layer's weights; tn: A stored [k][m], the weight gradient), bf16 / fp32 / int8, 1 to 4096 rows, inner and
           outer extents of 16 to 4096, multiples of 64, of 8 or odd; nt in bf16 also with the following bias + relu
           statement and a bf16 output;
  conv     NHWC convolutions, bf16 / fp32 / int8, 1x1 to 7x7 filters, stride 1 and 2, 3 to 256 channels, images of 7 to
           224 pixels; bf16 also with the following bias + relu statement and a bf16 output;
  window   max and average pooling and depthwise convolution, fp32 (max also bf16), 2x2 to 5x5, stride 1 and 2;
  upconv   stride-2 transposed convolutions (the data gradient of a strided convolution), fp32 and bf16.

Inputs are drawn on the GPU from the seed: activations N(0,1) (after a relu where a network has one), weights scaled by
their fan-in, int8 over its whole range.
"""
from __future__ import annotations

import math

import torch

from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W

_TORCH = {"i8": torch.int8, "i32": torch.int32, "bf16": torch.bfloat16, "f32": torch.float32}
_BYTES = {"i8": 1, "i32": 4, "bf16": 2, "f32": 4}


def _matmul(name, M, N, K, dtype, layout, fused=False):
    return dict(name=name, kind="matmul", M=M, N=N, K=K, dtype=dtype, layout=layout, fused=fused)


def _conv(name, N, H, Ci, Co, R, stride, dtype, fused=False):
    return dict(name=name, kind="conv", N=N, H=H, Ci=Ci, Co=Co, R=R, stride=stride, dtype=dtype, fused=fused)


def _window(name, op, N, H, C, R, stride, dtype="f32"):
    return dict(name=name, kind="window", op=op, N=N, H=H, C=C, R=R, stride=stride, dtype=dtype)


def _upconv(name, N, H, Ci, Co, R, dtype):
    return dict(name=name, kind="upconv", N=N, H=H, Ci=Ci, Co=Co, R=R, dtype=dtype)


def listed():
    return [
        # the smallest call: one small convolution of the repository's first configuration; launch and host time
        _conv("conv_tiny_f32", 1, 16, 8, 16, 3, 1, "f32"),
        # a Linear layer at a small batch (token by token inference): the weights are read once, few rows to share them
        _matmul("linear_decode_bf16", 8, 4096, 4096, "bf16", "nt", fused=True),
        # the repository's dense contraction: the largest product
        _matmul("matmul_bf16_4096", 4096, 4096, 4096, "bf16", "nn"),
        # a weight gradient X^T dY with extents that are no multiples of any tile
        _matmul("matmul_wgrad_bf16", 1000, 1000, 3000, "bf16", "tn"),
        # a single-precision product of an ordinary, untuned size
        _matmul("matmul_f32", 1000, 1000, 1000, "f32", "nn"),
        # a quantised Linear layer over 2000 rows
        _matmul("linear_i8", 2000, 2048, 2048, "i8", "nt"),
        # the repository's ResNet-style convolution
        _conv("conv3x3_bf16", 32, 56, 64, 64, 3, 1, "bf16"),
        # the first layer of an image network (three input channels) with its bias and relu
        _conv("conv7x7_rgb_bf16", 8, 224, 3, 64, 7, 2, "bf16", fused=True),
        # the repository's strided int8 convolution
        _conv("conv7x7_rgb_i8", 16, 224, 3, 64, 7, 2, "i8"),
        # the repository's pooling block
        _window("maxpool3x3s2_f32", "max", 32, 112, 64, 3, 2),
        # a depthwise layer on an odd image size
        _window("depthwise3x3_f32", "depthwise", 16, 57, 96, 3, 1),
        # the data gradient of a strided convolution
        _upconv("upconv3x3s2_f32", 8, 28, 32, 32, 3, "f32"),
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _extent(rng, lo, hi):
    """An extent spread over its logarithm: odd, a multiple of 8 or a multiple of 64."""
    grain = rng.choices([1, 8, 64], [3, 4, 5])[0]
    v = _log(rng, lo, hi)
    return min(hi, (v + grain - 1) // grain * grain)


_FLOP_CAP = {"bf16": 1.4e11, "i8": 1.7e10, "f32": 2.0e9}      # products: the listed ones' of each type


def draw(rng):
    kind = rng.choices(["matmul", "conv", "window", "upconv"], [5, 4, 2, 1])[0]
    while True:
        if kind == "matmul":
            dtype = rng.choices(["bf16", "f32", "i8"], [6, 2, 2])[0]
            layout = rng.choices(["nn", "nt", "tn"], [3, 4, 2])[0]
            c = _matmul("", _log(rng, 1, 4096), _extent(rng, 16, 4096), _extent(rng, 16, 4096), dtype, layout,
                        fused=dtype == "bf16" and layout == "nt" and rng.random() < 0.5)
            ok = 2.0 * c["M"] * c["N"] * c["K"] <= _FLOP_CAP[dtype]
        elif kind == "conv":
            dtype = rng.choices(["bf16", "f32", "i8"], [5, 2, 3])[0]
            R = rng.choice([1, 3, 3, 5, 7])
            Ci = 3 if rng.random() < 0.2 else _extent(rng, 8, 256)
            c = _conv("", _log(rng, 1, 32), _log(rng, 7, 224), Ci, _extent(rng, 8, 256), R, rng.choice([1, 1, 2]), dtype,
                      fused=dtype == "bf16" and rng.random() < 0.5)
            w = work(c)
            ok = w["bytes"] <= 1.3e8 and w["flops"] <= (2.0e9 if dtype == "f32" else 8.0e9)
        elif kind == "window":
            op = rng.choice(["max", "max", "avg", "depthwise"])
            c = _window("", op, _log(rng, 1, 32), _log(rng, 8, 112), _extent(rng, 3, 256), rng.choice([2, 3, 3, 5]), rng.choice([1, 2]),
                        "bf16" if op == "max" and rng.random() < 0.3 else "f32")
            ok = work(c)["bytes"] <= 1.3e8
        else:
            c = _upconv("", _log(rng, 1, 8), _log(rng, 7, 56), _extent(rng, 8, 64), _extent(rng, 8, 64), rng.choice([2, 3, 4]),
                        rng.choice(["f32", "f32", "bf16"]))
            ok = work(c)["flops"] <= 1.2e8
        if ok:
            del c["name"]
            return c


# ------------------------------------------------------------------ shapes
def _pad(c):
    return 0 if c["R"] == 2 else c["R"] // 2


def _out(c):
    if c["kind"] == "upconv":
        return 2 * (c["H"] - 1) + c["R"]
    return (c["H"] + 2 * _pad(c) - c["R"]) // c["stride"] + 1


def _taps(c):
    """In-image taps of all output positions along one direction."""
    p = _pad(c)
    return sum(1 for y in range(_out(c)) for i in range(c["R"]) if 0 <= c["stride"] * y + i - p < c["H"])


def _acc(dtype):
    return "i32" if dtype == "i8" else "f32"


def _out_dtype(c):
    if c.get("fused"):
        return "bf16"
    return c["dtype"] if c["kind"] == "window" else _acc(c["dtype"])


def _block(c):
    kind, dt = c["kind"], c["dtype"]
    if kind == "matmul":
        M, N, K = c["M"], c["N"], c["K"]
        if c["fused"]:
            return W.linear_bias_relu_program(M, N, K, "bf16", b_transposed=True)
        if c["layout"] == "tn":
            bufs = [W.Buffer("A", "in", dt, (K, M)), W.Buffer("B", "in", dt, (K, N)), W.Buffer("C", "out", _acc(dt), (M, N))]
            return W.flat_block(bufs, dict(m=M, n=N, k=K), [(["k", "m"], "assign"), (["k", "n"], "assign"), (["m", "n"], "add")])
        return W.matmul_block(M, N, K, dt, _acc(dt), b_transposed=c["layout"] == "nt")
    N, H, R = c["N"], c["H"], c["R"]
    if kind == "conv":
        if c["fused"]:
            return W.conv_bias_relu_program(N, H, H, c["Ci"], c["Co"], R, R, c["stride"], _pad(c), "bf16", "bf16")
        return W.conv2d_block(N, H, H, c["Ci"], c["Co"], R, R, c["stride"], _pad(c), dt, _acc(dt))
    if kind == "window":
        if c["op"] == "max":
            return W.maxpool_block(N, H, H, c["C"], R, c["stride"], _pad(c), dt)
        if c["op"] == "avg":
            return W.avgpool_block(N, H, H, c["C"], R, c["stride"], _pad(c), dt)
        return W.depthwise_conv_block(N, H, H, c["C"], R, R, c["stride"], _pad(c), dt)
    Ho = _out(c)
    bufs = [W.Buffer("I", "in", dt, (N, H, H, c["Ci"])), W.Buffer("F", "in", dt, (R, R, c["Ci"], c["Co"])),
            W.Buffer("O", "out", "f32", (N, Ho, Ho, c["Co"]))]
    return W.flat_block(bufs, dict(n=N, y=H, x=H, i=R, j=R, c=c["Ci"], k=c["Co"]),
                        [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", "2*y + i", "2*x + j", "k"], "add")])


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = c["dtype"]

    def normal(shape, scale=1.0, relu=False, dtype=dt):
        if dtype == "i8":
            return torch.randint(-128, 128, shape, generator=g, dtype=torch.int8, device="cuda")
        x = torch.randn(shape, generator=g, dtype=torch.float32, device="cuda")
        if relu:
            x = torch.relu(x)
        return (x * scale).to(_TORCH[dtype])

    if c["kind"] == "matmul":
        M, N, K = c["M"], c["N"], c["K"]
        a = normal((K, M) if c["layout"] == "tn" else (M, K))
        b = normal((N, K) if c["layout"] == "nt" else (K, N), (1.0 / K) ** 0.5 if c["fused"] else 1.0)
        return [a, b] + ([normal((N,), dtype="f32")] if c["fused"] else [])
    N, H, R = c["N"], c["H"], c["R"]
    if c["kind"] == "window":
        x = normal((N, H, H, c["C"]))
        if c["op"] == "max":
            return [x]
        if c["op"] == "avg":
            return [x, torch.full((1,), 1.0 / (R * R), dtype=_TORCH[dt], device="cuda")]
        return [x, normal((R, R, c["C"]), (1.0 / (R * R)) ** 0.5)]
    x = normal((N, H, H, c["Ci"]), relu=c["kind"] == "conv" and c["Ci"] > 3)      # an image is not the output of a relu
    if c["kind"] == "upconv":
        return [x, normal((R, R, c["Ci"], c["Co"]), (1.0 / (R * R * c["Co"])) ** 0.5)]
    f = normal((R, R, c["Co"], c["Ci"]), (2.0 / (R * R * c["Ci"])) ** 0.5)
    return [x, f] + ([normal((c["Co"],), 0.1, dtype="f32")] if c["fused"] else [])


# ------------------------------------------------------------------ what is measured
def prepare(case, seed):
    """The planned block, its inputs and its output buffer, as a program keeps them from call to call."""
    blk = _block(case)
    inputs = _inputs(case, seed)
    out = torch.zeros(blk.refs[-1].sizes, dtype=_TORCH[blk.refs[-1].dtype], device="cuda")
    return {"block": B.StripeBlock(blk), "inputs": inputs, "out": out}


def run(state):
    state["block"].run(state["inputs"], state["out"])
    return state["out"]


def work(case):
    """Each input and output once; two operations per point inside the image (pooling: one)."""
    c, kind = case, case["kind"]
    e, eo = _BYTES[c["dtype"]], _BYTES[_out_dtype(c)]
    if kind == "matmul":
        M, N, K = c["M"], c["N"], c["K"]
        return {"bytes": e * (M * K + K * N) + eo * M * N + (4 * N if c["fused"] else 0), "flops": 2.0 * M * N * K}
    N, H, Ho, R = c["N"], c["H"], _out(c), c["R"]
    if kind == "window":
        flops = float(N * c["C"] * _taps(c) ** 2) * (2.0 if c["op"] == "depthwise" else 1.0)
        return {"bytes": e * N * H * H * c["C"] + eo * N * Ho * Ho * c["C"] + (e * R * R * c["C"] if c["op"] == "depthwise" else 0), "flops": flops}
    taps = H * R if kind == "upconv" else _taps(c)
    return {"bytes": e * (N * H * H * c["Ci"] + R * R * c["Ci"] * c["Co"]) + eo * N * Ho * Ho * c["Co"] + (4 * c["Co"] if c.get("fused") else 0),
            "flops": 2.0 * N * taps * taps * c["Ci"] * c["Co"]}


def tolerance(case):
    """Integers and maxima are exact.  Float sums: products of bf16 values are exact in fp32 and every path accumulates in
    fp32, so what differs is the rounding of the sums, which grows with the square root of their length; a bf16 output adds
    its own rounding.  Measured against the same blocks in 64 bits: up to 8e-7, and 1.7e-3 with a bf16 output; four times that
    is allowed."""
    if case["dtype"] == "i8" or case.get("op") == "max":
        return "exact"
    if _out_dtype(case) == "bf16":
        return {"rel": 7e-3}
    return {"rel": 4e-6}


# ------------------------------------------------------------------ the same results in 64 bits
def exact(case, seed):
    """What `run` returns, as plain torch gives it in 64 bits: one product or one elementwise pass per filter tap.  The sums of
    the int8 cases stay below 2^53, so they are exact too."""
    c = case
    ins = [t.double() for t in _inputs(c, seed)]
    if c["kind"] == "matmul":
        a = ins[0].t().contiguous() if c["layout"] == "tn" else ins[0]
        b = ins[1].t().contiguous() if c["layout"] == "nt" else ins[1]
        y = a @ b
        return torch.relu(y + ins[2]) if c["fused"] else y
    N, H, R, Ho = c["N"], c["H"], c["R"], _out(c)
    x = ins[0]
    if c["kind"] == "upconv":
        y = x.new_zeros((N, Ho, Ho, c["Co"]))
        for i in range(R):
            for j in range(R):
                y[:, i:i + 2 * H - 1:2, j:j + 2 * H - 1:2] += x @ ins[1][i, j]
        return y
    p, s = _pad(c), c["stride"]
    lowest = c["kind"] == "window" and c["op"] == "max"
    x = torch.nn.functional.pad(x, (0, 0, p, p, p, p), value=float("-inf") if lowest else 0.0)
    y = None
    for i in range(R):
        for j in range(R):
            v = x[:, i:i + s * (Ho - 1) + 1:s, j:j + s * (Ho - 1) + 1:s]
            if c["kind"] == "conv":
                v = v.contiguous() @ ins[1][i, j].t().contiguous()
            elif c["op"] == "depthwise":
                v = v * ins[1][i, j]
            elif c["op"] == "avg":
                v = v * ins[1]
            y = v if y is None else torch.maximum(y, v) if lowest else y + v
    return torch.relu(y + ins[2]) if c.get("fused") else y
