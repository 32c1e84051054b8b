"""What is measured of this library: the calls a program makes that keeps a network's weights compressed.

Such a program decodes weights at inference time (whole sets, single layers, large matrices), convolves straight
from compressed weights, compresses weights that live on the GPU (tables and container), and dequantises symbols
it has decoded before.  Shapes are those of the ResNet-18 / ResNet-50 convolutions and of a 4096 x 11008 linear
stack; symbols follow the distributions the quantisers leave (mass on the zero-point; Laplace for linear layers).
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2406_06237_amd import binding as B

DEV = "cuda:0"

# conv1, then per stage and block the convolutions in the order a forward pass meets them:
# (output channels, input channels, kernel, stride, input height = width)


def _resnet18():
    out, size, cin = [(64, 3, 7, 2, 224)], 56, 64
    for stage, cout in enumerate((64, 128, 256, 512)):
        for block in range(2):
            stride = 2 if block == 0 and stage else 1
            out.append((cout, cin, 3, stride, size))
            out.append((cout, cout, 3, 1, size // stride))
            if cin != cout:
                out.append((cout, cin, 1, stride, size))
            size //= stride
            cin = cout
    return out


def _resnet50():
    out, size, cin = [(64, 3, 7, 2, 224)], 56, 64
    for stage, (width, blocks) in enumerate(((64, 3), (128, 4), (256, 6), (512, 3))):
        for block in range(blocks):
            stride = 2 if block == 0 and stage else 1
            out.append((width, cin, 1, 1, size))
            out.append((width, width, 3, stride, size))
            out.append((4 * width, width, 1, 1, size // stride))
            if block == 0:
                out.append((4 * width, cin, 1, stride, size))
            size //= stride
            cin = 4 * width
    return out


def _peaked(alphabet, z, p0):
    """P(z) = p0, the rest a two-sided geometric tail with ratio 1/2."""
    w = 0.5 ** np.abs(np.arange(alphabet) - z).astype(np.float64)
    w[z] = 0.0
    p = (1.0 - p0) * w / w.sum()
    p[z] = p0
    return p


def _laplace(alphabet, z, bits):
    """A Laplace distribution around z with an entropy of `bits` (or the most the alphabet allows)."""
    lo, hi = 1e-2, 1e3
    for _ in range(60):
        mid = math.sqrt(lo * hi)
        p = np.exp(-np.abs(np.arange(alphabet) - z) / mid)
        p /= p.sum()
        h = -(p[p > 0] * np.log2(p[p > 0])).sum()
        lo, hi = (mid, hi) if h < bits else (lo, mid)
    return p


def listed():
    return [
        # one small layer decoded when it is needed (a 64 x 64 1 x 1 convolution): launch and latency
        {"name": "decode_small_layer", "kind": "decode", "net": "layers", "layers": 1, "symbols": 4096, "bitwidth": 4, "dist": "peaked",
         "level": 0.8, "table_log": 10, "streams": 64, "chunk": 4096, "dtype": "f32", "channel_len": 0, "planned": False},
        # a 64 x 64 3 x 3 layer as a single stream: the container with the least framing, the longest chain
        {"name": "decode_one_stream", "kind": "decode", "net": "layers", "layers": 1, "symbols": 36864, "bitwidth": 4, "dist": "laplace",
         "level": 1.2, "table_log": 10, "streams": 1, "chunk": 36864, "dtype": "f32", "channel_len": 0, "planned": False},
        # all convolutions of a ResNet-18 / ResNet-50, decoded at every inference from arrays that stay: planned once
        {"name": "decode_resnet18", "kind": "decode", "net": "resnet18", "dist": "laplace", "table_log": 11, "streams": 32,
         "chunk": 16384, "dtype": "bf16", "planned": True},
        {"name": "decode_resnet50", "kind": "decode", "net": "resnet50", "dist": "peaked", "table_log": 12, "streams": 64,
         "chunk": 65536, "dtype": "bf16", "planned": True},
        # one block of a linear stack (4 matrices of 4096 x 4096, 3 of 4096 x 11008), a scale per output channel
        {"name": "decode_linear_block", "kind": "decode", "net": "linear", "layers": 7, "rows": 4096, "cols": 4096, "wide": 11008,
         "level": 2.5, "table_log": 12, "streams": 64, "chunk": 262144, "dtype": "bf16", "planned": False},
        # the convolution with decoding inside: one image through a late 3 x 3 layer (latency), and, at batch 64,
        # the 1 x 1 and 3 x 3 layers most of a ResNet-50 consists of
        {"name": "conv_3x3_one_image", "kind": "conv", "batch": 1, "size": 7, "cin": 512, "cout": 512, "k": 3, "stride": 1, "pad": 1,
         "x": "nhwc", "y": "nhwc", "dtype": "f32", "bitwidth": 5, "level": 0.9},
        {"name": "conv_1x1", "kind": "conv", "batch": 64, "size": 14, "cin": 1024, "cout": 256, "k": 1, "stride": 1, "pad": 0,
         "x": "c8", "y": "c8", "dtype": "bf16", "bitwidth": 4, "level": 0.85},
        {"name": "conv_3x3", "kind": "conv", "batch": 64, "size": 28, "cin": 128, "cout": 128, "k": 3, "stride": 1, "pad": 1,
         "x": "c8", "y": "c8", "dtype": "bf16", "bitwidth": 4, "level": 0.85},
        # every convolution of a ResNet-50, one call each, on 16 images
        {"name": "conv_resnet50", "kind": "conv_net", "batch": 16},
        # weights compressed on the GPU: decode tables and container of a ResNet-50, and of one late layer
        {"name": "compress_resnet50", "kind": "compress", "net": "resnet50", "dist": "peaked", "table_log": 12, "streams": 64, "chunk": 65536},
        {"name": "compress_layer", "kind": "compress", "net": "layers", "layers": 1, "symbols": 2359296, "bitwidth": 4, "dist": "laplace",
         "level": 1.6, "table_log": 11, "streams": 64, "chunk": 16384},
        # symbols that are in memory already (a 4096 x 11008 matrix) to weights, a scale per output channel
        {"name": "dequantise_matrix", "kind": "dequant", "symbols": 45088768, "channel_len": 11008, "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "decode", "conv", "conv", "conv", "compress", "compress", "dequant"))
    if kind in ("decode", "compress"):
        layers = _log_int(rng, 1, 48)
        case = {"kind": kind, "net": "layers", "layers": layers, "symbols": max(1000, _log_int(rng, 4096, 40e6) // layers),
                "bitwidth": rng.randint(2, 8), "dist": rng.choice(("peaked", "laplace")), "table_log": rng.randint(9, 12),
                "streams": rng.choice((64, 64, 32, 64, 48, 17)), "chunk": 16 * _log_int(rng, 128, 4096)}
        case["level"] = round(rng.uniform(0.55, 0.95) if case["dist"] == "peaked" else rng.uniform(0.8, 3.0), 3)
        if kind == "decode":
            case["dtype"] = rng.choice(("bf16", "bf16", "f32", "u8"))
            case["planned"] = rng.random() < 0.6
            case["channel_len"] = rng.choice((0, 0, 9 * rng.randint(8, 512)))
            if rng.random() < 0.1:
                case.update(layers=1, symbols=rng.randint(2000, 36864), streams=1, chunk=36864)
        return case
    if kind == "dequant":
        return {"kind": kind, "symbols": _log_int(rng, 4096, 45088768), "channel_len": rng.choice((0, rng.randint(64, 11008))),
                "dtype": rng.choice(("bf16", "bf16", "f32"))}
    k = rng.choice((1, 1, 3, 3, 7))
    size = rng.randint(6, 56)
    if k == 7:
        size, cin, cout = 2 * rng.randint(32, 112), 3, 64
    elif k == 3:
        cin, cout = 8 * rng.randint(4, 64), 16 * rng.randint(2, 32)
        if rng.random() < 0.7:
            cin = max(64, cin // 64 * 64)
    else:
        cin, cout = 8 * rng.randint(4, 256), 16 * rng.randint(2, 128)
        if rng.random() < 0.7:
            cin = max(64, cin // 64 * 64)
    stride = 2 if k == 7 else rng.choice((1, 1, 1, 2))
    out = (size - 1) // stride + 1
    batch = min(64, max(1, int(26e9 / (2.0 * out * out * cout * cin * k * k))))       # about the cost of the listed layers at most
    batch = _log_int(rng, 1, batch)
    layout = "nhwc" if cin % 8 else rng.choice(("c8", "c8", "nhwc"))
    return {"kind": "conv", "batch": batch, "size": size, "cin": cin, "cout": cout, "k": k, "stride": stride, "pad": k // 2,
            "x": layout, "y": rng.choice(("c8", "nhwc")) if cin % 8 else layout, "dtype": rng.choice(("bf16", "bf16", "f32")),
            "bitwidth": rng.randint(2, 8), "level": round(rng.uniform(0.6, 0.95), 3)}


# ---- inputs

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _symbols(pmf, n, gen):
    """n symbols drawn from pmf, a uint8 tensor on the GPU."""
    cdf = torch.from_numpy(np.cumsum(pmf)[:-1].astype(np.float32)).to(DEV)
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    for at in range(0, n, 1 << 25):
        m = min(1 << 25, n - at)
        out[at:at + m] = torch.bucketize(torch.rand(m, generator=gen, device=DEV), cdf, right=True, out_int32=True).to(torch.uint8)
    return out


class _Layer:
    def __init__(self, symbols, z, scale, bitwidth, channel_len, channel_scales, shape):
        self.symbols, self.z, self.scale, self.bitwidth = symbols, z, scale, bitwidth
        self.channel_len, self.channel_scales, self.shape = channel_len, channel_scales, shape


def _layers(case, seed):
    """The layers of a decode, compress or conv_net case: symbols on the GPU and their quantisers."""
    rng, gen = random.Random(seed), _generator(seed)
    net = case["net"]
    if net == "linear":
        shapes = [(case["rows"], case["cols"] if i < 4 else case["wide"], 1) for i in range(case["layers"])]
    elif net == "layers":
        shapes = [(1, case["symbols"] - (i * 37) % 256, 1) for i in range(case["layers"])]      # ragged sizes
    else:
        shapes = [s[:3] for s in (_resnet18() if net == "resnet18" else _resnet50())]
    sizes = [o * i * k * k for o, i, k in shapes]
    rank = np.empty(len(sizes), int)
    rank[np.argsort(sizes, kind="stable")] = np.arange(len(sizes))
    p0 = sorted(rng.uniform(0.7, 0.95) for _ in sizes)                # the largest layers are compressed hardest
    out = []
    for i, n in enumerate(sizes):
        if net == "linear":
            b, pmf = 4, _laplace(16, 8, case["level"])
        elif net == "layers":
            b = case["bitwidth"]
            pmf = (_peaked if case["dist"] == "peaked" else _laplace)(1 << b, 1 << (b - 1), case["level"])
        elif net == "resnet18":
            b = rng.randint(2, 6)
            pmf = _laplace(1 << b, 1 << (b - 1), rng.uniform(0.6, min(2.0, 0.9 * b)))
        else:
            b = rng.randint(1, 8)
            pmf = _peaked(1 << b, 1 << (b - 1), p0[rank[i]])
        clen = shapes[i][1] if net == "linear" else case.get("channel_len", 0)
        scales = None
        if clen:
            scales = (0.005 + 0.045 * torch.rand(-(-n // clen), generator=gen, device=DEV)).float()
        out.append(_Layer(_symbols(pmf, n, gen), 1 << (b - 1), float(np.float32(rng.uniform(0.005, 0.05))), b, clen, scales, shapes[i]))
    return out


def _activations(n, gen):
    return torch.randn(n, generator=gen, device=DEV, dtype=torch.float32).to(torch.bfloat16)


def _conv_layers(case, seed):
    """(layers, geometry) of a conv or conv_net case; geometry: (cout, cin, k, stride, pad, input size) per layer."""
    if case["kind"] == "conv_net":
        geo = [(o, i, k, s, k // 2, size) for o, i, k, s, size in _resnet50()]
        return _layers({"net": "resnet50"}, seed), geo
    gen, rng = _generator(seed), random.Random(seed)
    o, i, k, b = case["cout"], case["cin"], case["k"], case["bitwidth"]
    z = 1 << (b - 1)
    lay = _Layer(_symbols(_peaked(1 << b, z, case["level"]), o * i * k * k, gen), z, float(np.float32(rng.uniform(0.005, 0.05))), b, 0, None, (o, i, k))
    return [lay], [(o, i, k, case["stride"], case["pad"], case["size"])]


def _conv_inputs(case, seed, geo):
    """The activations: one buffer, of which every layer takes as much as it needs from the start."""
    return _activations(max(case["batch"] * size * size * cin for _, cin, _, _, _, size in geo), _generator(seed + 1))


def _conv_layouts(case, cin):
    if case["kind"] == "conv":
        return case["x"], case["y"]
    return ("c8" if cin % 8 == 0 else "nhwc"), "c8"


def prepare(case, seed):
    kind = case["kind"]
    if kind == "dequant":
        gen = _generator(seed)
        n, clen = case["symbols"], case["channel_len"]
        scales = (0.005 + 0.045 * torch.rand(-(-n // clen), generator=gen, device=DEV)).float() if clen else None
        return {"kind": kind, "symbols": _symbols(_laplace(16, 8, 2.5), n, gen), "channel_len": clen, "scales": scales, "dtype": case["dtype"]}
    if kind in ("conv", "conv_net"):
        layers, geo = _conv_layers(case, seed)
        host, first, rows = B.pack_conv_layers([l.symbols.cpu().numpy() for l in layers], [(o, i, k, k) for o, i, k, _, _, _ in geo], 12, 64,
                                               [l.z for l in layers], [l.scale for l in layers], [l.bitwidth for l in layers])
        d = B.to_device(host, DEV)
        xbuf = _conv_inputs(case, seed, geo)
        calls, ys = [], []
        for n, (cout, cin, k, stride, pad, size) in enumerate(geo):
            b, out = case["batch"], (size + 2 * pad - k) // stride + 1
            xl, yl = _conv_layouts(case, cin)
            x = xbuf[:b * size * size * cin].view((b, cin // 8, size, size, 8) if xl == "c8" else (b, size, size, cin))
            y = torch.empty(B.conv_out_shape(b, out, out, cout, yl), dtype=torch.float32 if case.get("dtype") == "f32" else torch.bfloat16, device=DEV)
            calls.append(B.conv_args(d, n, first[n], rows[n], x, (cout, cin, k, k), stride, pad, y, xl, yl))
            ys.append(y)
        return {"kind": kind, "container": d, "x": xbuf, "calls": calls, "y": ys}
    layers = _layers(case, seed)
    if kind == "decode":
        host = B.pack_layers([l.symbols.cpu().numpy() for l in layers], case["table_log"], case["streams"], case["chunk"],
                             [l.z for l in layers], [l.scale for l in layers], [l.bitwidth for l in layers],
                             [l.channel_len for l in layers],
                             [None if l.channel_scales is None else l.channel_scales.cpu().numpy() for l in layers], case["dtype"])
        d = B.to_device(host, DEV)
        out = B.alloc_out(d)
        args = B.decode_args(d, out)
        return {"kind": kind, "container": d, "out": out[:host.numel], "args": args,
                "plan": B.plan_decode(args, DEV) if case["planned"] else None}
    freqs = np.stack([B.normalize_freqs(torch.bincount(l.symbols, minlength=256).cpu().numpy(), case["table_log"]) for l in layers])
    return {"kind": kind, "symbols": torch.cat([l.symbols for l in layers]), "sizes": [l.symbols.numel() for l in layers],
            "freqs": torch.from_numpy(freqs.astype(np.int32)).to(DEV), "table_log": case["table_log"], "streams": case["streams"],
            "chunk": case["chunk"]}


def run(state):
    kind = state["kind"]
    if kind == "decode":
        if state["plan"] is None:
            B.decode_raw(state["args"], DEV)
        else:
            B.decode_planned_raw(state["args"], state["plan"], DEV)
        return {"weights": state["out"], "status": state["container"].status}
    if kind in ("conv", "conv_net"):
        for a in state["calls"]:
            B.conv_fused_raw(a, DEV)
        return state["y"]
    if kind == "compress":
        tables = B.build_tables_device(state["freqs"], state["table_log"])
        if len(state["sizes"]) == 1:
            packed = B.pack_layer_device(state["symbols"], state["freqs"], state["table_log"], state["streams"], state["chunk"])
        else:
            packed = B.pack_layers_device(state["symbols"], state["sizes"], state["freqs"], state["table_log"], state["streams"], state["chunk"])
        return {"tables": tables, "chunks": packed[0], "headers": packed[1], "words": packed[2], "used": packed[3], "status": packed[4]}
    return B.dequant_zp(state["symbols"], 8, 0.0125, state["dtype"], state["channel_len"], state["scales"])


def _numel(case):
    if case["net"] == "layers":
        return sum(case["symbols"] - (i * 37) % 256 for i in range(case["layers"]))
    if case["net"] == "linear":
        return case["rows"] * (4 * case["cols"] + (case["layers"] - 4) * case["wide"])
    return sum(o * i * k * k for o, i, k, _, _ in (_resnet18() if case["net"] == "resnet18" else _resnet50()))


def work(case):
    """Bytes: compressed words at the distributions' rate and their headers, weights or activations; operations: the
    convolutions' multiplications and additions, or one look-up's worth per symbol."""
    kind = case["kind"]
    size_of = {"u8": 1, "bf16": 2, "f32": 4}
    if kind == "dequant":
        return {"bytes": case["symbols"] * (1 + size_of[case["dtype"]]), "flops": 2 * case["symbols"]}
    if kind in ("conv", "conv_net"):
        geo = [(o, i, k, s, k // 2, z) for o, i, k, s, z in _resnet50()] if kind == "conv_net" else \
            [(case["cout"], case["cin"], case["k"], case["stride"], case["pad"], case["size"])]
        nbytes = flops = 0
        for cout, cin, k, stride, pad, size in geo:
            out = (size + 2 * pad - k) // stride + 1
            # a 1 x 1 kernel with a stride reads only the pixels it lands on; weights at about a bit and a half each
            seen = out if k == 1 else size
            nbytes += case["batch"] * (seen * seen * cin * 2 + out * out * cout * size_of[case.get("dtype", "bf16")]) + cout * cin * k * k * 3 // 16
            flops += 2 * case["batch"] * out * out * cout * cin * k * k
        return {"bytes": nbytes, "flops": flops}
    n = _numel(case)
    if case["net"] == "layers" and case["dist"] == "peaked":
        p = _peaked(1 << case["bitwidth"], 1 << (case["bitwidth"] - 1), case["level"])
        bits = -(p[p > 0] * np.log2(p[p > 0])).sum()
    else:
        bits = {"resnet18": 1.3, "resnet50": 0.7}.get(case["net"], case.get("level"))
    nbytes = n * bits / 8 + 4 * case["streams"] * n / case["chunk"]
    tables = case.get("layers", 53 if case["net"] == "resnet50" else 20) << case["table_log"]
    if kind == "decode":
        return {"bytes": int(nbytes + n * size_of[case["dtype"]] + tables * 16), "flops": 2 * n}
    return {"bytes": int(nbytes + n + tables * 32), "flops": 2 * n}


def tolerance(case):
    # Decoded weights are one rounding of an exact product, compressed words and tables are whole numbers: bit for bit.
    if case["kind"] not in ("conv", "conv_net"):
        return "exact"
    # Products are exact in fp32 (8-bit integers times bf16); the sums of up to 4608 of them are fp32 in any order (steps
    # of 32 added forwards and backwards: 4e-8 apart, and up to 4e-7 of the rms or of the value).
    if case.get("dtype") == "f32":
        return {"rel": 2e-7, "max": 2e-6}
    # The same sums rounded to bf16: where two orders straddle a rounding boundary, a value moves by one bf16 step, up to
    # 2^-7 of itself (3e-6 of the norm for those two orders; more values near a boundary on denser layers).
    return {"rel": 4e-5, "max": 8e-3}


def exact(case, seed):
    kind = case["kind"]
    if kind == "compress":
        return None
    if kind == "dequant":
        s = prepare(case, seed)
        q = s["symbols"].double() - 8.0
        if not case["channel_len"]:
            return q * float(np.float32(0.0125))
        return q * s["scales"].double().repeat_interleave(case["channel_len"])[:q.numel()]
    if kind == "decode":
        out = []
        for l in _layers(case, seed):
            if case["dtype"] == "u8":
                out.append(l.symbols)
            else:
                scale = l.scale if not l.channel_len else l.channel_scales.double().repeat_interleave(l.channel_len)[:l.symbols.numel()]
                out.append((l.symbols.double() - l.z) * scale)
        return {"weights": torch.cat(out), "status": None}
    layers, geo = _conv_layers(case, seed)
    xbuf = _conv_inputs(case, seed, geo)
    b, ys = case["batch"], []
    for lay, (cout, cin, k, stride, pad, size) in zip(layers, geo):
        out = (size + 2 * pad - k) // stride + 1
        xl, yl = _conv_layouts(case, cin)
        x = xbuf[:b * size * size * cin]
        x = x.view(b, cin // 8, size, size, 8).permute(0, 2, 3, 1, 4).reshape(b, size, size, cin) if xl == "c8" else x.view(b, size, size, cin)
        x = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
        w = ((lay.symbols.double() - lay.z) * lay.scale).view(cout, k, k, cin)
        y = torch.zeros(b * out * out, cout, dtype=torch.float64, device=DEV)
        for r in range(k):
            for s in range(k):
                tap = x[:, r:r + (out - 1) * stride + 1:stride, s:s + (out - 1) * stride + 1:stride, :]
                y += tap.reshape(-1, cin) @ w[:, r, s, :].t().contiguous()
        y = y.view(b, out, out, cout)
        ys.append(y.view(b, out, out, cout // 8, 8).permute(0, 3, 1, 2, 4).contiguous() if yl == "c8" else y)
    return ys
