"""The work that users of libdsqconv have it do, as measurable cases.

Four kinds of case, all through the public calls of ``binding``:

layer   one quantized convolution on its own: ``dsq_quantize_act`` of a float tensor, ``dsq_conv2d``
        to a float tensor (a network whose other operators run in floating point).
net     the quantized part of a network at inference: segments of layers whose codes are handed on by
        ``dsq_conv2d_requant`` (folded batch normalisation and ReLU in it), each segment beginning with
        ``dsq_quantize_act`` and ending with ``dsq_conv2d`` where the network needs floats (a residual
        sum, a pooling, a depthwise convolution).
wq      one layer with quantized weights and float activations (``dsq_conv2d_wq``).
soft    the training-mode quantizer of one tensor, forward and backward.

Weights are packed once in ``prepare``, as a program does when it loads its model.
"""
import math

import torch

from paper_1908_05033_amd import binding as B
from paper_1908_05033_amd import inputs

# Largest sizes of a drawn case: tensors of the largest layer of the VGG-16 stack at batch 32, and
# multiply-accumulates that keep a drawn case below that whole stack.
MAX_ELEMENTS = 32 * 64 * 224 * 224
MAX_MACS = 60e9
MAX_WQ_MACS = 8e9


def listed():
    return [
        # One image through one small layer: the shortest call there is, launches and latency.
        dict(name="image.64-64@32", kind="layer", N=1, C=64, H=32, W=32, K=64, R=3, stride=1, bits=4,
             layout="NHWC", signed=False),
        # One image through the deepest ResNet-18 layer (a single-image latency table's last row).
        dict(name="image.512-512@7", kind="layer", N=1, C=512, H=7, W=7, K=512, R=3, stride=1, bits=2,
             layout="NHWC", signed=False),
        # An ordinary layer at an ordinary batch.
        dict(name="layer.256-256@14", kind="layer", N=32, C=256, H=14, W=14, K=256, R=3, stride=1, bits=4,
             layout="NHWC", signed=False),
        # A strided layer whose tensors are in PyTorch's own layout on both sides.
        dict(name="layer.nchw.128-256@28", kind="layer", N=64, C=128, H=28, W=28, K=256, R=3, stride=2, bits=3,
             layout="NCHW", signed=False),
        # The largest tensors of the VGG-16 stack at batch 32.
        dict(name="layer.64-64@224", kind="layer", N=32, C=64, H=224, W=224, K=64, R=3, stride=1, bits=2,
             layout="NHWC", signed=False),
        # Whole networks, their layers chained where the network allows it.
        dict(name="net.vgg16.n32.2bit", kind="net", net="vgg16", N=32, hw=224, bits=2),
        dict(name="net.resnet18.n64.4bit", kind="net", net="resnet18", N=64, hw=56, bits=4),
        # Inverted bottlenecks: the narrow tensor has no ReLU, so its clip range starts below zero.
        dict(name="net.mobilenetv2.n64.4bit", kind="net", net="mobilenetv2", N=64, hw=56, bits=4),
        # The fully connected head of VGG-16 at a serving batch.
        dict(name="net.head.n64.4bit", kind="net", net="head", N=64, hw=1, bits=4),
        # 1-bit weights, float activations.
        dict(name="wq.128-128@28", kind="wq", N=64, C=128, H=28, W=28, K=128, R=3, stride=1, bits=1,
             layout="NHWC"),
        # A training step's quantizer: an activation tensor, and one layer's weights.
        dict(name="soft.activation", kind="soft", n=64 * 64 * 56 * 56, bits=2),
        dict(name="soft.weight", kind="soft", n=256 * 256 * 3 * 3, bits=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "net", "net", "net", "wq", "soft"])
    if kind == "soft":
        return dict(kind="soft", n=_log(rng, 20_000, MAX_ELEMENTS // 4), bits=rng.choice([1, 2, 3, 4]))
    if kind == "net":
        net = rng.choice(["vgg16", "resnet18", "mobilenetv2", "head"])
        hw = {"vgg16": rng.randint(112, 224), "resnet18": rng.randint(28, 64),
              "mobilenetv2": rng.randint(28, 64), "head": 1}[net]
        top = {"vgg16": 32, "resnet18": 64, "mobilenetv2": 64, "head": 256}[net]
        # the listed network cases bound the drawn ones' pixels
        pixels = {"vgg16": 32 * 224 * 224, "resnet18": 64 * 56 * 56, "mobilenetv2": 64 * 56 * 56, "head": 256}[net]
        N = max(1, min(_log(rng, 1, top), pixels // (hw * hw)))
        return dict(kind="net", net=net, N=N, hw=hw, bits=rng.choice([2, 3, 4]))
    while True:
        R = rng.choice([1, 3, 3])
        c = dict(kind=kind, N=_log(rng, 1, 64), C=_log(rng, 16, 512), H=_log(rng, 7, 224), W=0, K=_log(rng, 16, 512),
                 R=R, stride=rng.choice([1, 1, 2]), bits=rng.choice([1, 2] if kind == "wq" else [1, 2, 2, 3, 4, 4]),
                 layout=rng.choice(["NHWC", "NHWC", "NCHW"]))
        c["W"] = max(7, c["H"] + rng.choice([0, 0, rng.randint(-6, 6)]))
        if kind == "layer":
            c["signed"] = rng.random() < 0.25
        L = _layer_of(c)
        most, elements = (MAX_WQ_MACS, MAX_ELEMENTS // 8) if kind == "wq" else (MAX_MACS, MAX_ELEMENTS)
        if kind == "layer" and (c["signed"] or c["layout"] == "NCHW"):
            most, elements = most / 4, elements // 4
        if L["macs"] <= most and max(L["in"], L["out"]) <= elements:
            return c


# ---- networks: lists of segments, a segment a list of layers -----------------------------------
# A layer is (C_in, C_out, R, stride, ends): `ends` says what its outputs are: "codes" (handed to the
# next layer after batch normalisation and ReLU), "signed" (the same without ReLU) or "float".

def _segments(net, hw):
    """[(H, signed input, [layers], shortcut or None)]"""
    if net == "vgg16":
        out = [(hw, False, [(64, 64, 3, 1, "float")], None)]
        for h, ci, co, n in ((hw // 2, 64, 128, 2), (hw // 4, 128, 256, 3), (hw // 8, 256, 512, 3),
                             (hw // 16, 512, 512, 3)):
            chans = [ci] + [co] * n
            out.append((h, False, [(chans[i], chans[i + 1], 3, 1, "codes" if i + 1 < n else "float")
                                   for i in range(n)], None))
        return out
    if net == "resnet18":
        out, h, ci = [], hw, 64
        for co in (64, 128, 256, 512):
            for block in range(2):
                s = 2 if co != ci else 1
                out.append((h, False, [(ci, co, 3, s, "codes"), (co, co, 3, 1, "float")],
                            (ci, co, 1, s, "float") if s == 2 else None))
                h, ci = (h - 1) // s + 1, co
        return out
    if net == "mobilenetv2":
        return [(hw, False, [(144, 24, 1, 1, "signed"), (24, 144, 1, 1, "float")], None),
                (hw // 4, False, [(576, 96, 1, 1, "signed"), (96, 576, 1, 1, "float")], None),
                (hw // 8, True, [(320, 1280, 1, 1, "float")], None)]
    return [(1, False, [(25088, 4096, 1, 1, "codes"), (4096, 4096, 1, 1, "float")], None)]


def _layer_of(c):
    p = (c["R"] - 1) // 2
    Ho, Wo = (c["H"] + 2 * p - c["R"]) // c["stride"] + 1, (c["W"] + 2 * p - c["R"]) // c["stride"] + 1
    return {"pad": p, "Ho": Ho, "Wo": Wo, "in": c["N"] * c["C"] * c["H"] * c["W"], "out": c["N"] * c["K"] * Ho * Wo,
            "macs": c["N"] * Ho * Wo * c["K"] * c["C"] * c["R"] ** 2}


def _net_layers(case):
    """Every layer of a network case as a dict with its geometry, in order, with its segment's number
    and place ("first" reads the segment's codes, "next" the previous layer's, "shortcut" the segment's)."""
    for s, (h, signed, layers, shortcut) in enumerate(_segments(case["net"], case["hw"])):
        hin = h
        for i, (ci, co, R, stride, ends) in enumerate(layers):
            c = dict(N=case["N"], C=ci, H=h, W=h, K=co, R=R, stride=stride, bits=case["bits"])
            yield s, "first" if i == 0 else "next", signed, ends, c
            h = _layer_of(c)["Ho"]
            signed = ends == "signed"
        if shortcut:
            ci, co, R, stride, ends = shortcut
            yield s, "shortcut", False, ends, dict(N=case["N"], C=ci, H=hin, W=hin, K=co, R=R, stride=stride,
                                                   bits=case["bits"])


# ---- inputs --------------------------------------------------------------------------------------

def _range(bits, signed):
    """A learned clip range of a unit-variance activation tensor: the 99.5th percentile of |N(0, 1)| at
    one and two bits, the 99.9th above; about symmetric where the tensor has both signs."""
    u = 2.807 if bits <= 2 else 3.2905
    return (-0.93 * u, u) if signed else (0.0, u)


def _activation(shape, signed, g):
    x = torch.randn(shape, generator=g, device="cuda")
    return x if signed else x.abs_()


def _pack(c, g, weight_only=False):
    """Packed He-normal weights of a layer, and the side table."""
    w = torch.randn((c["K"], c["C"], c["R"], c["R"]), generator=g, device="cuda") * math.sqrt(2.0 / (c["C"] * c["R"] ** 2))
    flat = w.reshape(c["K"], -1)
    if weight_only and c["bits"] == 1:
        u_w = flat.abs().mean(dim=1)
        l_w = -u_w
    elif c["bits"] <= 2:
        l_w, u_w = flat.amin(dim=1), flat.amax(dim=1)
    else:
        u_w = 3.0 * flat.std(dim=1)
        l_w = -u_w
    bits_field = 4 if weight_only else c["bits"]
    packed = torch.empty(B.dsq_wgt_packed_bytes(c["K"], c["C"], c["R"], c["R"], bits_field), dtype=torch.uint8, device="cuda")
    aux = torch.empty(B.dsq_wgt_aux_bytes(c["K"], c["R"], c["R"]), dtype=torch.uint8, device="cuda")
    B.dsq_pack_weights_for(w, l_w.contiguous(), u_w.contiguous(), None, c["K"], c["C"], c["R"], c["R"], c["bits"], bits_field,
                           packed, aux)
    return packed, aux


def _codes(N, H, W, C, bits):
    return (torch.empty(B.dsq_act_packed_bytes(N, H, W, C, bits), dtype=torch.uint8, device="cuda"),
            torch.empty(N * H * W, dtype=torch.int32, device="cuda"))


def _desc(c):
    return B.make_desc(c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["R"], c["stride"], (c["R"] - 1) // 2, c["bits"])


def _shaped(N, H, W, C, layout):
    return (N, C, H, W) if layout == "NCHW" else (N, H, W, C)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(inputs.BASE_SEED + int(seed))
    if case["kind"] == "soft":
        n = case["n"]
        return {"kind": "soft", "x": torch.randn(n, generator=g, device="cuda") * 0.78, "gy": torch.randn(n, generator=g, device="cuda"),
                "y": torch.empty(n, device="cuda"), "gx": torch.empty(n, device="cuda"),
                "g3": torch.empty(3, dtype=torch.float64, device="cuda"), "bits": case["bits"]}
    if case["kind"] == "net":
        return _prepare_net(case, int(seed), g)
    L = _layer_of(case)
    layout = B.DSQ_NCHW if case["layout"] == "NCHW" else B.DSQ_NHWC
    s = {"kind": case["kind"], "c": case, "desc": _desc(case), "layout": layout,
         "x": _activation(_shaped(case["N"], case["H"], case["W"], case["C"], case["layout"]), case.get("signed", False), g),
         "out": torch.empty(_shaped(case["N"], L["Ho"], L["Wo"], case["K"], case["layout"]), device="cuda")}
    s["w"], s["aux"] = _pack(case, g, case["kind"] == "wq")
    if case["kind"] == "layer":
        s["range"] = _range(case["bits"], case["signed"])
        s["codes"], s["sums"] = _codes(case["N"], case["H"], case["W"], case["C"], case["bits"])
    return s


def _prepare_net(case, seed, g):
    segments, last, out_signed = [], None, False
    for n, (seg, place, signed, ends, c) in enumerate(_net_layers(case)):
        L = _layer_of(c)
        if place == "first":
            codes, sums = _codes(c["N"], c["H"], c["W"], c["C"], c["bits"])
            segments.append({"x": _activation((c["N"], c["H"], c["W"], c["C"]), signed, g), "geom": (c["N"], c["C"], c["H"], c["W"]),
                             "range": _range(c["bits"], signed), "codes": codes, "sums": sums, "layers": []})
            last = (codes, sums, segments[-1]["range"])
        src = (segments[-1]["codes"], segments[-1]["sums"], segments[-1]["range"]) if place == "shortcut" else last
        layer = {"desc": _desc(c), "codes": src[0], "sums": src[1], "range": src[2], "ends": ends}
        layer["w"], layer["aux"] = _pack(c, g)
        if ends == "float":
            layer["out"] = torch.empty((c["N"], L["Ho"], L["Wo"], c["K"]), device="cuda")
        else:
            scale, shift = inputs.affine_params(seed * 100 + n, c["K"])
            layer["scale"], layer["shift"] = torch.from_numpy(scale).cuda(), torch.from_numpy(shift).cuda()
            layer["next"] = _range(c["bits"], ends == "signed")
            layer["codes_next"], layer["sums_next"] = _codes(c["N"], L["Ho"], L["Wo"], c["K"], c["bits"])
            last = (layer["codes_next"], layer["sums_next"], layer["next"])
        segments[-1]["layers"].append(layer)
    return {"kind": "net", "bits": case["bits"], "segments": segments}


# ---- one pass ------------------------------------------------------------------------------------

def run(s):
    if s["kind"] == "layer":
        c, (l, u) = s["c"], s["range"]
        B.dsq_quantize_act(s["x"], s["layout"], c["N"], c["C"], c["H"], c["W"], l, u, c["bits"], s["codes"], s["sums"])
        B.dsq_conv2d(s["desc"], s["codes"], s["sums"], l, u, s["w"], s["aux"], s["out"], s["layout"])
        return s["out"]
    if s["kind"] == "wq":
        B.dsq_conv2d_wq(s["desc"], s["x"], s["layout"], s["w"], s["aux"], s["out"], s["layout"])
        return s["out"]
    if s["kind"] == "soft":
        B.dsq_soft_quantize_fwd(s["x"], -1.0, 1.0, 0.2, s["bits"], s["y"])
        B.dsq_soft_quantize_bwd(s["x"], s["gy"], -1.0, 1.0, 0.2, s["bits"], s["gx"], s["g3"])
        return {"y": s["y"], "grad_x": s["gx"], "grad_alpha_l_u": s["g3"]}
    got = []
    for seg in s["segments"]:
        N, C, H, W = seg["geom"]
        B.dsq_quantize_act(seg["x"], B.DSQ_NHWC, N, C, H, W, seg["range"][0], seg["range"][1], s["bits"], seg["codes"], seg["sums"])
        for y in seg["layers"]:
            if y["ends"] == "float":
                B.dsq_conv2d(y["desc"], y["codes"], y["sums"], y["range"][0], y["range"][1], y["w"], y["aux"], y["out"], B.DSQ_NHWC)
                got.append(y["out"])
            else:
                B.dsq_conv2d_requant(y["desc"], y["codes"], y["sums"], y["range"][0], y["range"][1], y["w"], y["aux"], y["scale"],
                                     y["shift"], y["ends"] == "codes", y["next"][0], y["next"][1], s["bits"], y["codes_next"],
                                     y["sums_next"])
                got += [y["codes_next"], y["sums_next"]]
    return got


# ---- what a pass cannot do without ---------------------------------------------------------------

def _weight_bytes(c):
    """Weight codes at their own width, and the side table's step, level and code sum per channel."""
    return c["K"] * c["C"] * c["R"] ** 2 * c["bits"] / 8 + 12 * c["K"]


def work(case):
    if case["kind"] == "soft":
        return {"bytes": 16 * case["n"], "flops": 40 * case["n"]}      # x, grad_y in; y, grad_x out
    if case["kind"] != "net":
        L = _layer_of(case)
        return {"bytes": 4 * (L["in"] + L["out"]) + _weight_bytes(case), "flops": 2 * L["macs"]}
    total, flops = 0, 0
    for seg, place, signed, ends, c in _net_layers(case):
        L = _layer_of(c)
        total += _weight_bytes(c) + (4 * L["in"] if place == "first" else 0)
        # a chained layer's codes and code sums are results as well
        total += 4 * L["out"] if ends == "float" else L["out"] * c["bits"] / 8 + 4 * L["out"] / c["K"] + 8 * c["K"]
        flops += 2 * L["macs"]
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # Four times what the path differs by from itself in 64 bits (torch float64, measured):
    # layer and net: the sums are exact and rounded once (2.5e-8, largest 6e-8); codes are exact.
    # wq: sums of up to 4608 products in 32 bits (7.2e-7, largest 5.4e-6).
    # soft: tanh and its derivatives in 32 bits (9.3e-7, largest 3.3e-6).
    if case["kind"] == "wq":
        return {"rel": 3e-6, "max": 2.2e-5}
    if case["kind"] == "soft":
        return {"rel": 4e-6, "max": 1.4e-5}
    return {"rel": 1e-7, "max": 2.5e-7}
