"""The calls whose speed counts: fused tile execution of convolution / max-pool
stacks through ``mafat.Plan`` and ``mafat.Network``.

Sizes are those of this repository's workloads, tests and benchmark (YOLOv2's
first 16 layers at 608x608 and 416x416, the tiny stack, the strided and
padded stem, the VGG-style stack, single layers), with odd extents and other
batches among them; every execution the plan offers is there (all tiles at
once, one tile at a time, tile rows with reuse, the stage partition; KRSC and
packed weights; float32 and bfloat16).

A case: ``net`` (a stack below, or ``first:last`` of it after an ``@``, or
layers spelled out, see ``_layers``), the input ``h``, ``w``, ``c``, ``batch``,
``dtype``, the ``tiling`` in the paper's notation, ``mode`` (how tiles run) and
``packed`` (weights repacked once, as a serving program does).
"""
import math

import numpy as np
import torch

from paper_2107_06960_amd import mafat as M
from paper_2107_06960_amd import workloads as W

# 3x3 convolutions in pairs and triples between pools, linear last layer.
VGG_LIKE = [W.conv(64), W.conv(64), W.maxpool(), W.conv(128), W.conv(128), W.maxpool(),
            W.conv(256), W.conv(256), W.conv(256, act=W.LINEAR)]
NETS = {"yolo": W.YOLOV2_16, "tiny": W.TINY, "stem": W.OTHER_CNN, "vgg": VGG_LIKE}
MODES = {"all": {}, "part": {"stage_partition": True}, "rows": {"row_reuse": True}, "seq": {"tile_batch": 1}}


def _case(net, h, w, c, batch, dtype, tiling, mode="all", packed=False, name=None):
    d = {"net": net, "h": h, "w": w, "c": c, "batch": batch, "dtype": dtype, "tiling": tiling, "mode": mode,
         "packed": packed}
    return dict(d, name=name) if name else d


def listed():
    return [
        # The smallest call: three layers on a thumbnail, two launches; latency and host work.
        _case("tiny", 64, 64, 3, 1, "f32", "2x2/NoCut", name="tiny_f32"),
        # The benchmark: one camera frame through both groups, every tile at once.
        _case("yolo", 608, 608, 3, 1, "bf16", "5x5/8/2x2", packed=True, name="yolo608_bf16"),
        # Throughput: a batch of eight frames, the largest call.
        _case("yolo", 608, 608, 3, 8, "bf16", "4x4/12/1x1", packed=True, name="yolo608_b8_bf16"),
        # Full precision: the paper's data type, one fused group on a 3x3 grid.
        _case("yolo", 416, 416, 3, 1, "f32", "3x3/NoCut", name="yolo416_f32"),
        # Little memory: the shallow group, tile rows in order, overlaps kept.
        _case("yolo@0:8", 608, 608, 3, 1, "bf16", "5x5/NoCut", "rows", True, name="shallow_rows_bf16"),
        # Least memory: the same group in the paper's order, one tile after another.
        _case("yolo@0:8", 608, 608, 3, 1, "bf16", "5x5/NoCut", "seq", True, name="shallow_seq_bf16"),
        # The deep group alone on a batch of cut tensors, stage by stage, weights as a framework stores them.
        _case("yolo@8:16", 76, 76, 128, 4, "bf16", "2x2/NoCut", "part", name="deep_part_bf16"),
        # Other networks: strided and padded layers (7x7/2, 3x3/2, 5x5, pools of three kinds), a small batch.
        _case("stem", 224, 200, 3, 4, "bf16", "2x3/4/2x2", name="stem_bf16"),
        # The same kind of stack in float32, one frame, one fused group.
        _case("stem", 224, 200, 3, 1, "f32", "3x3/NoCut", name="stem_f32"),
        # 3x3 convolutions without a first-layer pool on odd extents, three groups.
        _case("vgg", 131, 97, 3, 2, "f32", "3x2/3/2x3/6/1x2", name="vgg_f32"),
        # One wide layer on a ragged tensor, not tiled: what a program calls layer by layer.
        _case("c512f3s1p1", 37, 41, 256, 2, "bf16", "1x1/NoCut", name="layer3x3_bf16"),
        # A padded pool on its own: bound by memory.
        _case("m3s2p1", 112, 112, 64, 8, "bf16", "1x1/NoCut", name="pool_bf16"),
    ]


def draw(rng):
    """One more case: a network, a group of it, or a single layer, of any size up to the listed ones."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    for _ in range(1000):
        kind = rng.choice(["yolo", "yolo", "shallow", "deep", "stem", "vgg", "conv", "conv", "pool"])
        dtype = rng.choice(["bf16", "f32"])
        mode = rng.choice(["all", "all", "part", "rows", "seq"])
        packed = rng.random() < 0.5
        batch = rng.choice([1, 1, 2, 3, 4, 8])
        g = lambda hi: "%dx%d" % (rng.randint(1, hi), rng.randint(1, hi))  # noqa: E731
        if kind == "yolo":
            h, c, net = log(96, 608), 3, "yolo"
            tiling = rng.choice([g(3) + "/NoCut", g(5) + "/8/" + g(2), g(4) + "/12/" + g(2), g(5) + "/4/" + g(2)])
        elif kind == "shallow":
            h, c, net, tiling = log(64, 608), 3, "yolo@0:8", g(5) + "/NoCut"
        elif kind == "deep":
            h, c, net, tiling = log(13, 76), 128, "yolo@8:16", g(3) + "/NoCut"
        elif kind == "stem":
            h, c, net, tiling = log(97, 224), 3, "stem", rng.choice([g(3) + "/NoCut", g(3) + "/4/" + g(2)])
        elif kind == "vgg":
            h, c, net, tiling = log(48, 224), 3, "vgg", g(3) + "/3/" + g(3) + "/6/" + g(2)
        elif kind == "conv":
            f, s = rng.choice([(1, 1), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2), (1, 2)])
            c = rng.choice([3, 16, 32, 48, 64, 96, 128, 256, 512])
            h, tiling = log(9, 152), g(3) + "/NoCut"
            net = "c%df%ds%dp%d" % (rng.choice([16, 24, 32, 64, 96, 128, 256, 512]), f, s, (f - 1) // 2)
        else:
            f, s, p = rng.choice([(2, 2, 0), (3, 2, 1), (3, 1, 1), (3, 2, 0)])
            h, c, tiling, net = log(16, 224), rng.choice([16, 24, 64, 128, 256]), g(3) + "/NoCut", "m%ds%dp%d" % (f, s, p)
        w = max(9, int(h * rng.uniform(0.7, 1.0)))
        case = _case(net, h, w, c, batch, dtype, tiling, mode, packed)
        # no more work than the listed cases of the same data type (and kind of layer) have,
        # and no more tiles than the listed one-tile-at-a-time one
        flops, launches = work(case)["flops"], 1
        if mode == "seq":
            launches = sum(r * q for r, q in zip(*W.parse_tiling(tiling, len(_layers(net)))[1:]))
        generic = any(L["op"] == W.CONV and (L["f"] > 3 or L["s"] > 1) for L in _layers(net))
        if flops > (2.7e9 if generic else 2e11 if dtype == "bf16" else 2.4e10) or launches > 25:
            continue
        if _fits(case):
            return case
    raise RuntimeError("no case drawn")


def _layers(net):
    """"yolo", "yolo@0:8", or layers spelled out: c<out>f<filter>s<stride>p<padding> and m<window>s<stride>p<padding>."""
    name, _, part = net.partition("@")
    if name in NETS:
        a, b = (int(v) for v in part.split(":")) if part else (0, len(NETS[name]))
        return NETS[name][a:b]
    out = []
    for t in net.split(","):
        head, p = t.split("p")
        head, s = head.split("s")
        if t[0] == "c":
            c_out, f = head[1:].split("f")
            out.append(W.conv(int(c_out), int(f), s=int(s), p=int(p)))
        else:
            out.append(W.maxpool(int(head[1:]), int(s), int(p)))
    return out


def _shapes(case):
    """Output (h, w, c) of every layer."""
    h, w, c = case["h"], case["w"], case["c"]
    out = []
    for L in _layers(case["net"]):
        h = (h + 2 * L["p"] - L["f"]) // L["s"] + 1
        w = (w + 2 * L["p"] - L["f"]) // L["s"] + 1
        c = L["c_out"] if L["op"] == W.CONV else c
        out.append((h, w, c))
    return out


def _group_ends(case):
    n = len(_layers(case["net"]))
    starts, rows, cols = W.parse_tiling(case["tiling"], n)
    return [s - 1 for s in starts[1:]] + [n - 1], rows, cols


def _fits(case):
    shapes = _shapes(case)
    if min(min(s) for s in shapes) < 1:
        return False
    ends, rows, cols = _group_ends(case)
    return all(r <= shapes[e][0] and q <= shapes[e][1] for e, r, q in zip(ends, rows, cols))


def work(case):
    """Input, parameters, cut tensors and output once; the multiply-adds of the layers on whole tensors (no tile computes
    another's halo)."""
    size = 2 if case["dtype"] == "bf16" else 4
    shapes, ends = _shapes(case), _group_ends(case)[0]
    data = case["h"] * case["w"] * case["c"] + sum(math.prod(shapes[e]) for e in ends)
    bytes_, flops, c = case["batch"] * data * size, 0, case["c"]
    for L, (h, w, co) in zip(_layers(case["net"]), shapes):
        if L["op"] == W.CONV:
            k = L["f"] * L["f"] * c
            bytes_ += co * k * size + 8 * co
            flops += 2 * h * w * co * k * case["batch"]
        else:
            flops += h * w * co * L["f"] * L["f"] * case["batch"]
        c = co
    return {"bytes": bytes_, "flops": flops}


def _inputs(case, seed):
    """(x on the GPU, parameters on the host), as the repository's workloads draw them: an image in [0, 1), or what a leaky
    layer leaves inside a network."""
    layers = _layers(case["net"])
    params = W.make_inputs(layers, 1, 1, case["c"], 1, seed, case["dtype"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["batch"], case["h"], case["w"], case["c"])
    if case["c"] == 3:
        x = torch.rand(shape, generator=gen, device="cuda")
    else:
        x = torch.nn.functional.leaky_relu(torch.randn(shape, generator=gen, device="cuda"), 0.1)
    return x.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32), params


def prepare(case, seed):
    """The plan, the device parameters and buffers a program keeps, and a frame (or a batch of frames) on the GPU."""
    x, params = _inputs(case, seed)
    plan = M.Plan(_layers(case["net"]), (case["h"], case["w"], case["c"]), case["tiling"],
                  packed_weights=case["packed"], **MODES[case["mode"]])
    return {"net": M.Network(plan, params, case["batch"], case["dtype"]), "x": x}


def run(state):
    net = state["net"]
    y = net.run(state["x"])
    return {"y": y, "cuts": list(net.cuts)}


def tolerance(case):
    """Relative 2-norm errors against 64 bits as measured: float32 3e-7 for one layer, 1.8e-6 after 16; bfloat16 1.7e-3 for one
    layer (its output's rounding), 6e-3 after 16.  Four times those.  A pool only selects."""
    layers = _layers(case["net"])
    convs = sum(L["op"] == W.CONV for L in layers)
    if convs == 0:
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1.5e-6 if convs == 1 else 7e-6}
    return {"rel": 7e-3 if convs == 1 else 2.4e-2}


def exact(case, seed):
    """The stack layer by layer in float64: a convolution as one matrix product per filter tap."""
    x, params = _inputs(case, seed)
    x = x.double()
    ends, cuts = _group_ends(case)[0], []
    for k, L in enumerate(_layers(case["net"])):
        f, s, p = L["f"], L["s"], L["p"]
        conv = L["op"] == W.CONV
        b, h, w, c = x.shape
        ho, wo = (h + 2 * p - f) // s + 1, (w + 2 * p - f) // s + 1
        pad = torch.full((b, h + 2 * p, w + 2 * p, c), 0.0 if conv else -math.inf, dtype=torch.float64, device=x.device)
        pad[:, p:p + h, p:p + w] = x
        y = None
        if conv:
            wt = torch.from_numpy(np.ascontiguousarray(params["w"][k])).to(x.device).double()
        for ky in range(f):
            for kx in range(f):
                t = pad[:, ky:ky + s * (ho - 1) + 1:s, kx:kx + s * (wo - 1) + 1:s]
                if conv:
                    t = t.reshape(-1, c) @ wt[:, ky, kx].t().contiguous()
                    y = t if y is None else y.add_(t)
                else:
                    y = t.clone() if y is None else torch.maximum(y, t)
        if conv:
            v = y * torch.from_numpy(params["scale"][k]).to(x.device).double()
            v += torch.from_numpy(params["bias"][k]).to(x.device).double()
            if L["act"] == W.LEAKY:
                v = torch.maximum(v, 0.1 * v)
            y = v.reshape(b, ho, wo, -1)
        x = y
        if k in ends:
            cuts.append(x)
    return {"y": cuts[-1], "cuts": cuts[:-1]}
