"""The convolutions this library's speed is judged on: 12 listed ones, and a generator of more of the same ranges.

One case is one convolution layer as an inference program calls it: the filter is packed, the zero row filled and the
indirection buffer built beforehand (`prepare`), and one pass is one call of the convolution on a device tensor
(`run`) -- or, where the image size changes from call to call, the rebuild of the indirection buffer and that call.

A case's keys: N, Hin, Win, C, K, R, S, stride, dilation, pad (the same on both axes), dtype ("bf16", "u8i8", "f32"),
zero_point (u8i8), fused (bias and ReLU in the output stage, bfloat16 or uint8 output), per_image (the
batch-independent indirection buffer), rebuild (the buffer is built in the pass), first (the input is an image and not
the output of a ReLU).
"""
import math

import torch
import torch.nn.functional as F

from paper_1907_02129_amd import binding as icv
from paper_1907_02129_amd.workloads import ConvShape


def _case(name, N, hw, C, K, k, *, stride=1, dilation=1, pad=0, dtype="bf16", zero_point=0, fused=False,
          per_image=False, rebuild=False, first=False):
    h, w = hw if isinstance(hw, tuple) else (hw, hw)
    c = dict(N=N, Hin=h, Win=w, C=C, K=K, R=k, S=k, stride=stride, dilation=dilation, pad=pad, dtype=dtype,
             zero_point=zero_point, fused=fused, per_image=per_image, rebuild=rebuild, first=first)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call there is: what a launch costs
        _case("tiny_f32", 1, 8, 4, 8, 3, pad=1, dtype="f32", first=True),
        # one image at a time, as an interactive service sees it: ResNet-18's last stage on a single 7 x 7 map
        _case("stage4_one_image", 1, 7, 512, 512, 3, pad=1, fused=True),
        # the same layer at a throughput batch: few output pixels, a long reduction
        _case("stage4_batch32", 32, 7, 512, 512, 3, pad=1),
        # the benchmark's headline: ResNet-18's first stage at batch 32, single-precision output
        _case("stage1_batch32", 32, 56, 64, 64, 3, pad=1),
        # a downsampling layer in a server whose batch size varies: the buffer that serves every batch, fused output
        _case("strided_per_image", 32, 56, 128, 256, 3, stride=2, pad=1, fused=True, per_image=True),
        # the largest: a dilated (segmentation) layer over a big offline batch
        _case("dilated_batch256", 256, 64, 128, 128, 3, dilation=2, pad=2),
        # quantised inference, layer to layer: uint8 in (ReLU in front: zero point 0), uint8 out
        _case("int8_to_uint8", 32, 28, 256, 256, 3, pad=1, dtype="u8i8", fused=True),
        # SqueezeNet's classifier: pointwise, 1000 output channels (ragged against every tile), 13 x 13 pixels
        _case("classifier_1x1", 32, 13, 512, 1000, 1),
        # the first layer of an image network, three channels stored in four
        _case("first_layer_bf16", 32, 224, 4, 64, 7, stride=2, pad=3, first=True),
        # the same layer in single precision on the image as it is, three channels
        _case("first_layer_rgb_f32", 16, 224, 3, 64, 7, stride=2, pad=3, dtype="f32", first=True),
        # SqueezeNet's fire6 at a large batch with its 48 channels stored as they are
        _case("fire6_c48", 128, 27, 48, 192, 3, pad=1, fused=True),
        # single precision, images of no regular size that changes from call to call: buffer build and convolution
        _case("resized_f32", 2, (45, 75), 64, 64, 3, pad=1, dtype="f32", rebuild=True),
    ]


def _out(c):
    f = lambda n: (n + 2 * c["pad"] - c["dilation"] * (c["R"] - 1) - 1) // c["stride"] + 1
    return f(c["Hin"]), f(c["Win"])


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Layer widths: most are multiples of 32 or powers of two, some multiples of 8, a few any number."""
    c, kind = _log(rng, lo, hi), rng.random()
    if kind < 0.45:
        return 1 << round(math.log2(c))
    if kind < 0.75:
        return max(32, round(c / 32) * 32)
    if kind < 0.93:
        return max(8, round(c / 8) * 8)
    return c


def draw(rng):
    while True:
        dtype = rng.choice(["bf16", "bf16", "bf16", "u8i8", "u8i8", "f32"])
        kind = rng.choice(["3x3", "3x3", "3x3", "1x1", "5x5", "first"])
        dilation, first = 1, kind == "first"
        if first:
            k, stride = rng.choice([3, 5, 7]), rng.choice([1, 2, 2])
            C = rng.choice([1, 3, 3, 4, 4, 4])
            h = _log(rng, 32, 256)
        else:
            k = int(kind[0])
            stride = rng.choice([1, 1, 1, 2])
            dilation = 2 if k == 3 and stride == 1 and rng.random() < 0.2 else 1
            C = _channels(rng, 16, 512)
            h = _log(rng, 7, 96)
        w = h if rng.random() < 0.6 else max(7, int(h * rng.uniform(0.6, 1.7)))
        pad = rng.choice([0, dilation * (k // 2)]) if rng.random() < 0.2 else dilation * (k // 2)
        c = _case("", _log(rng, 1, 256), (h, w), C, _channels(rng, 8, 1024 if k == 1 else 512), k, stride=stride,
                  dilation=dilation, pad=pad, dtype=dtype, fused=rng.random() < 0.5, per_image=rng.random() < 0.2,
                  rebuild=rng.random() < 0.15, first=first)
        if dtype == "u8i8":
            c["zero_point"] = 128 if first else rng.choice([0, 0, 0, 128, rng.randrange(256)])
        if min(_out(c)) < 1:
            continue
        # no more than the largest listed cases: the batch is cut until it fits, single precision and widths that are
        # no multiple of 64 earlier than the rest
        usual = c["C"] % 64 == 0 and dtype != "f32"
        most = 250e9 if usual else (3.5e9 if dtype == "f32" else 14e9)
        while c["N"] > 1 and (work(c)["flops"] > most or work(c)["bytes"] > 400e6):
            c["N"] -= max(1, c["N"] // 5)
        if work(c)["flops"] <= most and work(c)["bytes"] <= 400e6:
            return c


_SIZE = {"f32": 4, "bf16": 2, "u8i8": 1}


def work(c):
    Hout, Wout = _out(c)
    M, T = c["N"] * Hout * Wout, c["R"] * c["S"]
    size = _SIZE[c["dtype"]]
    out_size = {"f32": 2, "bf16": 2, "u8i8": 1}[c["dtype"]] if c["fused"] else 4
    # an indirection entry is an offset of four bytes; written by the pass that rebuilds the buffer, else read.  A
    # pointwise layer without stride or padding needs none
    entries = 0 if T == 1 and c["stride"] == 1 and c["pad"] == 0 else (Hout * Wout if c["per_image"] else M) * T * 4
    # the input pixels that a strided layer steps over are not read
    used_y, used_x = min(c["Hin"], Hout * c["R"]), min(c["Win"], Wout * c["S"])
    return {"bytes": c["N"] * used_y * used_x * c["C"] * size + c["K"] * T * c["C"] * size + M * c["K"] * out_size +
                     entries + (4 * c["K"] if c["fused"] else 0),
            "flops": 2.0 * M * c["K"] * T * c["C"]}


def tolerance(c):
    if c["dtype"] == "u8i8":
        return "exact"                       # integer sums, and one rounding that is fixed by the interface
    if c["fused"]:
        # bfloat16 output of single-precision sums: against sums in 64 bits, rounded, it differs by 1e-5 to 4e-5, by
        # one bfloat16 step (up to 2^-7) where a value lies near a tie
        return {"rel": 1.5e-4, "max": 1.6e-2}
    # single-precision sums: against sums in 64 bits they differ by 1e-8 to 7e-7, single values by up to 5e-6
    return {"rel": 3e-6, "max": 2e-5}


def prepare(c, seed):
    dev = "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    s = ConvShape("case", c["N"], c["Hin"], c["Win"], c["C"], c["K"], c["R"], c["S"], SY=c["stride"], SX=c["stride"],
                  DY=c["dilation"], DX=c["dilation"], PT=c["pad"], PL=c["pad"], PB=c["pad"], PR=c["pad"],
                  dtype=c["dtype"], zero_point=c["zero_point"])
    x = torch.randn((s.N, s.Hin, s.Win, s.C), generator=g, device=dev)
    w = torch.randn((s.K, s.R, s.S, s.C), generator=g, device=dev)
    red = math.sqrt(s.R * s.S * s.C)
    if c["first"] and s.C == 4:
        x[..., 3:] = 0                       # three channels stored in four
        w[..., 3:] = 0
    if not c["first"]:
        x = x.relu_()                        # every layer but the first reads what a ReLU left
    if s.dtype == "u8i8":
        x = (x * 48 + s.zero_point).round_().clamp_(0, 255).to(torch.uint8)
        w = (w * 32).round_().clamp_(-127, 127).to(torch.int8)
    else:
        t = torch.bfloat16 if s.dtype == "bf16" else torch.float32
        x, w = x.to(t), (w / red).to(t)
    buf = icv.prepare(s, w, plan=icv.PLAN_PER_IMAGE if c["per_image"] else 0)
    st = {"x": x, "w": w, "buf": buf, "rebuild": c["rebuild"], "ep": None}
    if c["fused"]:
        if s.dtype == "u8i8":
            st["bias"] = (torch.randn(s.K, generator=g, device=dev) * 500).round_().to(torch.int32)
            st["ep"] = icv.make_epilogue(st["bias"], relu=True, out_type=icv.ICV_OUT_U8,
                                         out_scale=1.0 / (24.0 * red), out_zero_point=0)
            out_type = torch.uint8
        else:
            st["bias"] = torch.randn(s.K, generator=g, device=dev) * 0.1
            st["ep"] = icv.make_epilogue(st["bias"], relu=True, out_type=icv.ICV_OUT_BF16)
            out_type = torch.bfloat16
        st["out"] = torch.empty(buf.output.shape, dtype=out_type, device=dev)
        buf.output = st["out"]
    return st


def run(st):
    buf = st["buf"]
    if st["rebuild"]:
        icv.setup_indirection(buf.p, buf.indirection)
    if st["ep"] is None:
        return icv.run(buf, st["x"])
    icv.conv2d_nhwc_fused(buf.p, st["x"], buf.packed, buf.indirection, buf.zero_row, st["ep"], st["out"])
    return st["out"]


def exact(c, seed):
    """The same convolution as one matrix product per kernel element in 64 bits.  Integers below 2^53 are exact there;
    the requantisation of a uint8 output is defined in single precision and is done in it."""
    st = prepare(c, seed)
    x, w = st["x"].double(), st["w"].double()
    zp = float(c["zero_point"]) if c["dtype"] == "u8i8" else 0.0
    (Hout, Wout), p, d, t = _out(c), c["pad"], c["dilation"], c["stride"]
    x = F.pad(x - zp, (0, 0, p, p, p, p))
    y = torch.zeros((c["N"] * Hout * Wout, c["K"]), dtype=torch.float64, device=x.device)
    for ky in range(c["R"]):
        for kx in range(c["S"]):
            rows = x[:, ky * d: ky * d + (Hout - 1) * t + 1: t, kx * d: kx * d + (Wout - 1) * t + 1: t]
            y.addmm_(rows.reshape(-1, c["C"]), w[:, ky, kx].t())
    y = y.view(c["N"], Hout, Wout, c["K"])
    if st["ep"] is not None:
        y = (y + st["bias"].double()).relu_()
        if c["dtype"] == "u8i8":
            return (y.float() * st["ep"].out_scale).round_().clamp_(0, 255).to(torch.uint8)
        return y
    return y.to(torch.int32) if c["dtype"] == "u8i8" else y
