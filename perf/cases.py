"""The layer workloads that the library's speed is judged by: the shapes of the benchmark
(workloads.py), one-image serving, ragged sizes, both tile sizes, both activation layouts, narrow
codes, weight-only quantization and the off-line filter transform, each through the entry points
a program calls.  All sizes are layer shapes; inputs and filters are seeded random draws with the
distributions of workloads.py."""
import math

import torch

from paper_2003_08646_amd import binding as B
from paper_2003_08646_amd import workloads as Wk
from paper_2003_08646_amd.layer import LanceConv

# What a case dict holds, with the value that most layers have.
_DEFAULTS = dict(kind="conv", plan="layer", n=1, c=64, k=64, h=32, w=32, pad=1, m=2, bits=8, bits_w=8,
                 layout="nchw", ranges="dynamic", packed=False, dist="relu_normal")


def _case(name=None, **kw):
    case = dict(_DEFAULTS, **kw)
    return case if name is None else dict(case, name=name)


def listed():
    """Twelve cases.  kind: "conv" the fused call, "weight_only" full-precision inputs on
    quantized filters, "filters" the off-line transform of the weights; plan: one "layer", or
    "vgg16", the thirteen 3x3 layers of a VGG-16-shaped network back to back."""
    return [
        # the smallest benchmark layer: one CIFAR image, a call bound by launches and latency
        _case("one_image_c16", n=1, c=16, k=16, h=32, w=32, dist="uniform01"),
        # one-image serving of the whole network with calibrated ranges (Sec. 3.4's inference mode)
        _case("net_one_image_static", plan="vgg16", n=1, h=224, w=224, ranges="static"),
        # the CIFAR-ResNet block layer at training-evaluation batch
        _case("resnet_block_c64", n=128, c=64, k=64, h=32, w=32),
        # mid-network layer, F(2x2) and F(4x4)
        _case("mid_c128_m2", n=64, c=128, k=128, h=56, w=56, m=2),
        _case("mid_c128_m4", n=64, c=128, k=128, h=56, w=56, m=4),
        # deep layer, many channels on small images
        _case("deep_c512", n=64, c=512, k=512, h=14, w=14),
        # the whole network at the benchmark's batch, ranges found in every call: the largest
        _case("net_batch16", plan="vgg16", n=16, h=224, w=224),
        # the paper's own activation layout
        _case("nhwc_c128", n=64, c=128, k=128, h=56, w=56, layout="nhwc"),
        # odd channel, filter and image sizes, no padding, calibrated ranges
        _case("ragged_m4_static", n=13, c=100, k=72, h=37, w=29, pad=0, m=4, ranges="static"),
        # the 4-4 rows: two codes to a byte, calibrated ranges
        _case("packed_w4_x4", n=64, c=512, k=512, h=14, w=14, bits=4, bits_w=4, packed=True,
              ranges="static"),
        # the 4-32 row: 4-bit filters on full-precision inputs, a CIFAR layer
        _case("weight_only_w4", kind="weight_only", n=32, c=64, k=64, h=32, w=32, bits_w=4),
        # loading a network: every layer's weights transformed and quantized once
        _case("filters_net", kind="filters", plan="vgg16", h=224, w=224),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case: a layer of any size up to the largest listed ones, most of them convolution
    calls, with pad 1, 8 bits, NCHW and dynamic ranges the commonest values of each option."""
    kind = rng.choices(("conv", "weight_only", "filters"), (80, 10, 10))[0]
    m = rng.choices((2, 4), (65, 35))[0]
    ranges = rng.choices(("dynamic", "static"), (60, 40))[0]
    if kind == "conv" and rng.random() < 0.12:
        size = 16 * rng.randint(2, 14)
        return _case(plan="vgg16", n=_log(rng, 1, 16), h=size, w=size, m=m, ranges=ranges,
                     bits_w=rng.choices((8, 6, 5, 4), (70, 10, 10, 10))[0])
    c, k = _log(rng, 3, 512), _log(rng, 8, 512)
    if rng.random() < 0.5:  # half of the layers have channel counts in steps of 16
        c, k = 16 * max(1, round(c / 16)), 16 * max(1, round(k / 16))
    if kind == "filters":
        return _case(kind=kind, c=c, k=k, m=m, bits_w=rng.choices((8, 6, 4), (60, 20, 20))[0])
    h = _log(rng, 7, 224)
    w = h if rng.random() < 0.6 else max(7, min(224, int(h * rng.uniform(0.7, 1.4))))
    pad = rng.choices((1, 0, 2), (80, 14, 6))[0]
    # a batch that keeps the layer below the largest listed single layer (for weight-only calls
    # below the listed one): operations of the direct convolution and elements of x and y
    ops, elements = (59e9, 25.7e6) if kind == "conv" else (2.5e9, 2.1e6)
    one = h * w * max(1, c * k) * 18
    most = int(min(128, ops / one, elements / (h * w * max(c, k))))
    if most < 1:
        h = w = int(min(math.sqrt(ops / (18 * c * k)), math.sqrt(elements / max(c, k))))
        most = 1
    n = _log(rng, 1, most)
    bits = rng.choices((8, 6, 4, 3), (72, 8, 14, 6))[0]
    bits_w = bits if rng.random() < 0.8 else rng.choice((8, 6, 5, 4))
    if kind == "weight_only":
        return _case(kind=kind, n=n, c=c, k=k, h=h, w=w, pad=pad, m=m,
                     bits_w=rng.choice((8, 6, 4, 4)))
    packed = bits <= 4 and bits_w <= 4 and c > 16 and rng.random() < 0.6
    layout = rng.choices(("nchw", "nhwc"), (75, 25))[0]
    return _case(n=n, c=c, k=k, h=h, w=w, pad=pad, m=m, bits=bits, bits_w=bits_w, layout=layout,
                 ranges=ranges, packed=packed, dist="normal" if c <= 4 else "relu_normal")


def _layers(case):
    """The layers of a case: one, or the network's thirteen at the case's image size."""
    if case["plan"] == "vgg16":
        return [L.with_(H=L.H * case["h"] // 224, W=L.W * case["w"] // 224, m=case["m"],
                        bits=case["bits"], bits_w=case["bits_w"])
                for L in Wk.vgg16_layers(case["n"])]
    return [Wk.Layer("layer", case["n"], case["c"], case["k"], case["h"], case["w"],
                     pad=case["pad"], m=case["m"], bits=case["bits"], bits_w=case["bits_w"],
                     x_dist=case["dist"])]


def _flags(case):
    return ((B.LANCE_LAYOUT_NHWC if case["layout"] == "nhwc" else 0) |
            (B.LANCE_INPUT_RANGE_STATIC if case["ranges"] == "static" else 0) |
            (B.LANCE_CODES_PACKED4 if case["packed"] else 0))


def _activations(layer, nhwc, gen):
    shape = (layer.N, layer.H, layer.W, layer.C) if nhwc else (layer.N, layer.C, layer.H, layer.W)
    if layer.x_dist == "uniform01":
        return torch.rand(shape, generator=gen, device="cuda")
    x = torch.randn(shape, generator=gen, device="cuda")
    return x.clamp_min_(0.0) if layer.x_dist == "relu_normal" else x


def _conv(layer, flags):
    return LanceConv(layer.N, layer.C, layer.H, layer.W, layer.K, layer.pad, layer.m, layer.bits,
                     flags=flags, bits_w=layer.bits_w)


def prepare(case, seed):
    """Layer objects with prepared filters (and calibrated ranges), and the activations."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, nhwc, flags = case["kind"], case["layout"] == "nhwc", _flags(case)
    if kind == "weight_only":
        flags &= ~B.LANCE_INPUT_RANGE_STATIC
    items = []
    for layer in _layers(case):
        weights = torch.randn((layer.K, layer.C, 3, 3), generator=gen, device="cuda")
        weights *= math.sqrt(2.0 / (9.0 * layer.C))
        conv = _conv(layer, flags)
        if kind == "filters":
            items.append((conv, weights))
            continue
        conv.prepare_filters(weights)
        if flags & B.LANCE_INPUT_RANGE_STATIC:
            # ranges of another batch of the same kind, as a calibration run finds them
            calibrate = _conv(layer, flags & ~B.LANCE_INPUT_RANGE_STATIC)
            calibrate.prepare_filters(weights)
            calibrate.forward(_activations(layer, nhwc, gen))
            conv.v_range.copy_(calibrate.v_range)
        items.append((conv, _activations(layer, nhwc, gen)))
    return dict(kind=kind, dynamic=case["ranges"] == "dynamic", items=items)


def run(state):
    """One pass: every layer's call, on the current stream."""
    if state["kind"] == "filters":
        for conv, weights in state["items"]:
            conv.prepare_filters(weights)
        return [(conv.uq, conv.u_range, conv.u_rowsum) for conv, _ in state["items"]]
    if state["kind"] == "weight_only":
        for conv, x in state["items"]:
            B.lance_conv3x3_winograd_wq_f32(conv.desc, x, conv.uq, conv.u_range, conv.y)
        return [conv.y for conv, _ in state["items"]]
    outputs = [conv.forward(x) for conv, x in state["items"]]
    if state["dynamic"]:  # the ranges the call found are an output too
        return [(y, conv.v_range) for y, (conv, _) in zip(outputs, state["items"])]
    return outputs


def work(case):
    """x and the prepared filters read, y written, once each; the multiply-adds of the
    (m+2)^2 products per tile, filter and channel.  Filter transform: weights read, codes and
    sums written, two small matrix products per filter and channel."""
    bytes_, flops = 0.0, 0.0
    for L in _layers(case):
        s = B.lance_query_sizes(B.make_desc(L.N, L.C, L.H, L.W, L.K, L.pad, L.m, L.bits,
                                            _flags(case) | B.LANCE_FILTER_BITS(L.bits_w)))
        prepared = s.uq_bytes + s.u_range_bytes + s.u_rowsum_bytes
        if case["kind"] == "filters":
            edge = L.m + 2
            bytes_ += L.K * L.C * 36 + prepared
            flops += L.K * L.C * 2 * (edge * 9 + edge * edge * 3)
            continue
        bytes_ += L.N * L.C * L.H * L.W * 4 + s.y_bytes + prepared
        flops += 2.0 * s.E * L.K * L.C * s.P
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Filter codes and sums are whole numbers and their ranges are minima and maxima: exact.
    The codes and integer products of a convolution are exact too; what is left is the binary32
    rounding of the de-quantization and of the output transform, whose terms cancel.  Against the
    same steps in binary64, over the listed cases and forty drawn ones: rel <= 1.5e-6, max <=
    1.7e-5 (F(4x4)); with packed codes, whose offset of 8 adds terms that cancel, 2.0e-5 and
    1.4e-4; weight-only 7e-7 and 1.2e-5.  Four times that."""
    if case["kind"] == "filters":
        return "exact"
    return {"rel": 8e-5, "max": 6e-4} if case["packed"] else {"rel": 6e-6, "max": 7e-5}
