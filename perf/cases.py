"""The work whose speed counts: what users of this library have it do, over the real range of sizes.

Five kinds of case:

  masks   one mask pyramid: the masks and kept lists of every resolution of a network from one input mask
  layer   one convolution through the one-call form (mask in, features out), or without a mask
  grouped one grouped convolution in its own form (weights of one group's channels only)
  step    a mask pyramid and four 3x3 layers that share its lists, recorded into a HIP graph once
          and replayed: how a serving loop runs a fixed set of layers
  stack   a whole network's convolutions through ConvStack.run

Inputs follow the paper's census: ReLU activations, and masks of few large regions with about half of
the pixels irrelevant.  The weights of a network belong to the network, not to an input: they are made
once per network and kept, as a program that serves it keeps them.
"""
import functools
import math

import torch

from paper_2207_10741_amd import binding as B
from paper_2207_10741_amd import synth, workloads
from paper_2207_10741_amd.stacks import ConvStack

DEVICE = "cuda:0"
DTYPES = {"f32": B.F32, "bf16": B.BF16, "f16": B.F16, "fp8": B.FP8}
BYTES = {"f32": 4, "bf16": 2, "f16": 2, "fp8": 1}
NETWORKS = {"resnet18": (workloads.resnet18, 3), "resnet50": (workloads.resnet50_bottlenecks, 64),
            "vgg16": (workloads.vgg16, 3), "mobilenetv2": (workloads.mobilenetv2, 3)}


def masks(name, n, h, w, levels=4, packed=False, irrelevant=0.48):
    return dict(name=name, kind="masks", n=n, h=h, w=w, levels=levels, packed=packed, irrelevant=irrelevant)


def layer(name, n, h, w, c_in, c_out, k=3, stride=1, dtype="bf16", out="same", masked=True, irrelevant=0.48):
    return dict(name=name, kind="layer", n=n, h=h, w=w, c_in=c_in, c_out=c_out, k=k, stride=stride, groups=1,
                dtype=dtype, out=out, masked=masked, irrelevant=irrelevant)


def grouped(name, n, h, w, channels, groups, dtype="bf16", masked=True, irrelevant=0.48):
    return dict(layer(name, n, h, w, channels, channels, dtype=dtype, masked=masked, irrelevant=irrelevant),
                kind="grouped", groups=groups)


def step(name, n, side, dtype="bf16", irrelevant=0.48):
    return dict(name=name, kind="step", n=n, side=side, dtype=dtype, irrelevant=irrelevant)


def stack(name, net, n, h, w, dtype="bf16", mask="objects", irrelevant=0.48, chain=False, compact=False, keep=False):
    return dict(name=name, kind="stack", net=net, n=n, h=h, w=w, dtype=dtype, mask=mask, irrelevant=irrelevant,
                chain=chain, compact=compact, keep=keep)


def listed():
    return [
        # one camera frame's mask for all resolutions of a classifier: a few microseconds, launches only
        masks("masks_1x224", 1, 224, 224),
        # one small layer on one image, the way the README shows it
        layer("layer_1x56_c64", 1, 56, 56, 64, 64),
        # a layer that fits no tile: odd image sides, channel counts off the tile sizes, stride 2, 16-bit floats
        layer("layer_ragged_f16", 3, 75, 101, 72, 200, stride=2, dtype="f16"),
        # the standard convolution (no mask) at a size that fills the chip
        layer("layer_dense_f16", 16, 60, 80, 256, 256, dtype="f16", masked=False),
        # fp32 storage: callers that cannot give up precision
        layer("layer_f32", 2, 60, 80, 64, 64, dtype="f32"),
        # the grouped 3x3 of a ResNeXt's first stage
        grouped("grouped_c128_g32", 16, 56, 56, 128, 32),
        # the benchmark's four ResNet-50 layers with their masks
        step("step_b16", 16, 128),
        # one image through a whole network, every feature map wanted: the latency case
        stack("resnet18_b1", "resnet18", 1, 224, 224, keep=True),
        # depthwise-separable blocks
        stack("mobilenetv2_b32", "mobilenetv2", 32, 224, 224, chain=True),
        # bottleneck blocks of VGA frames, kept rows handed on as lists; 16-bit and 8-bit storage
        stack("resnet50_b32", "resnet50", 32, 120, 160, chain=True, compact=True),
        stack("resnet50_fp8_b32", "resnet50", 32, 120, 160, dtype="fp8", chain=True),
        # full-HD frames with a depth threshold as mask, every feature map wanted and zero-filled: the largest
        stack("vgg16_hd_b8", "vgg16", 8, 1080, 1920, mask="depth", irrelevant=0.5, keep=True),
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["masks", "layer", "layer", "layer", "f32", "grouped", "step", "stack", "stack", "stack", "stack"])
    irr = round(rng.uniform(0.3, 0.7), 2)
    if kind == "masks":
        c = masks("", _log(rng, 1, 32), _log(rng, 64, 640), _log(rng, 64, 640), rng.choice([3, 4, 5]),
                  rng.random() < 0.3, irr)
    elif kind == "layer":
        dtype = rng.choice(["bf16", "bf16", "f16", "fp8"])
        unit = 16 if dtype == "fp8" else 8
        ci, co = unit * _log(rng, 2, 512 // unit), unit * _log(rng, 2, 512 // unit)
        k = rng.choice([1, 3, 3, 3, 5])
        n, h, w = _log(rng, 1, 32), _log(rng, 14, 160), _log(rng, 14, 160)
        while n > 1 and n * h * w * k * k * ci * co > 2e11:
            n //= 2
        c = layer("", n, h, w, ci, co, k, rng.choice([1, 1, 2]), dtype, rng.choice(["same", "same", "f32"]),
                  rng.random() < 0.75, irr)
    elif kind == "f32":
        n, h, w, ci, co = _log(rng, 1, 8), _log(rng, 14, 120), _log(rng, 14, 120), _log(rng, 16, 128), _log(rng, 16, 128)
        while n > 1 and n * h * w * 9 * ci * co > 4e9:
            n //= 2
        c = layer("", n, h, w, ci, co, dtype="f32", masked=rng.random() < 0.75, irrelevant=irr)
    elif kind == "grouped":
        groups = rng.choice([16, 32])
        c = grouped("", _log(rng, 2, 32), _log(rng, 7, 60), _log(rng, 7, 60), groups * rng.choice([4, 8, 16]), groups,
                    rng.choice(["bf16", "f16"]), rng.random() < 0.75, irr)
    elif kind == "step":
        c = step("", _log(rng, 2, 32), rng.randrange(56, 161), rng.choice(["bf16", "bf16", "f16", "fp8"]), irr)
    else:
        net = rng.choice(list(NETWORKS))
        chain = rng.random() < 0.6
        if net == "resnet18":
            c = stack("", net, _log(rng, 1, 8), rng.randrange(160, 321), rng.randrange(160, 321),
                      rng.choice(["bf16", "f16"]), irrelevant=irr, chain=chain, keep=not chain)
        elif net == "resnet50":
            c = stack("", net, _log(rng, 2, 32), rng.randrange(56, 121), rng.randrange(56, 161),
                      rng.choice(["bf16", "f16", "fp8"]), irrelevant=irr, chain=chain, compact=chain and rng.random() < 0.5,
                      keep=not chain)
        elif net == "vgg16":
            h = _log(rng, 224, 1080)
            c = stack("", net, _log(rng, 1, 6), h, h * 16 // 9, mask="depth", irrelevant=irr, chain=chain, keep=not chain)
        else:
            c = stack("", net, _log(rng, 2, 64), rng.randrange(160, 257), rng.randrange(160, 257),
                      rng.choice(["bf16", "f16"]), irrelevant=irr, chain=chain, keep=not chain)
    del c["name"]
    return c


# ---- inputs ------------------------------------------------------------------

def _activations(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE).relu_().to(B.torch_dtype(DTYPES[dtype]))


def _weights(gen, shape, fan_in, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE).mul_(math.sqrt(2.0 / fan_in)).to(B.torch_dtype(DTYPES[dtype]))


def _bias(gen, c):
    return torch.randn((c,), generator=gen, device=DEVICE).mul_(0.01)


def _mask(seed, n, h, w, irrelevant, kind="objects"):
    paint = synth.mask_depth_ramp if kind == "depth" else synth.mask_objects
    return torch.from_numpy(paint(n, h, w, irrelevant, seed)).to(DEVICE)


@functools.lru_cache(maxsize=2)
def _network(net, n, h, w, dtype):
    return ConvStack(NETWORKS[net][0](), n, h, w, DTYPES[dtype])


def _pyramid(mask, levels, packed=False):
    """The network's resolutions: the input's own, then one halving after another."""
    steps = [((3, 3), (1, 1), (1, 1), (1, 1))] + [((3, 3), (2, 2), (1, 1), (1, 1))] * (levels - 1)
    p = B.PreparedPyramid(mask, steps, packed=packed)
    for m_out, idx, count in p.levels:      # list entries past the count are nobody's: zero, not leftovers
        idx.zero_()
    return p


def _prepare_step(case, gen, seed):
    n, side, dtype = case["n"], case["side"], case["dtype"]
    mask = _mask(seed, n, side, side, case["irrelevant"])
    pyramid = _pyramid(mask, 4)
    calls, outs = [pyramid], []
    for (c, _), (_, h, w), (m_out, idx, count) in zip(workloads.sweep_shapes(), pyramid.dims, pyramid.levels):
        desc = B.conv_desc(n, h, w, c, c, in_dtype=DTYPES[dtype], flags=B.RELU)
        ws = B.ready_workspace(torch.empty((B.workspace_bytes(desc),), dtype=torch.uint8, device=DEVICE))
        call = B.PreparedConv(desc, _activations(gen, (n, h, w, c), dtype), _weights(gen, (c, 3, 3, c), 9 * c, dtype),
                              _bias(gen, c), mask_in=m_out, mask_out=m_out, idx=idx, count=count, workspace=ws,
                              workspace_ready=True)
        calls.append(call)
        outs.append(call.out)

    def once():
        for call in calls:
            call()

    once()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        once()
    torch.cuda.synchronize()
    return dict(kind="step", graph=graph, outs=outs, calls=calls)


def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    if kind == "step":
        return _prepare_step(case, gen, seed)
    n, h, w = case["n"], case["h"], case["w"]
    if kind == "masks":
        mask = _mask(seed, n, h, w, case["irrelevant"])
        return dict(kind=kind, pyramid=_pyramid(mask, case["levels"], case["packed"]))
    if kind == "stack":
        return dict(kind=kind, net=_network(case["net"], n, h, w, case["dtype"]),
                    x=_activations(gen, (n, h, w, NETWORKS[case["net"]][1]), case["dtype"]),
                    mask=_mask(seed, n, h, w, case["irrelevant"], case["mask"]),
                    chain=case["chain"], compact=case["compact"], keep=case["keep"])
    k, dtype, groups = case["k"], case["dtype"], case["groups"]
    ci, co = case["c_in"], case["c_out"]
    desc = B.conv_desc(n, h, w, ci, co, (k, k), (case["stride"],) * 2, (k // 2,) * 2, in_dtype=DTYPES[dtype],
                       out_dtype=B.F32 if case["out"] == "f32" else None, flags=B.RELU)
    return dict(kind=kind, desc=desc, groups=groups, x=_activations(gen, (n, h, w, ci), dtype),
                weights=_weights(gen, (co, k, k, ci // groups), k * k * ci // groups, dtype), bias=_bias(gen, co),
                mask=_mask(seed, n, h, w, case["irrelevant"]) if case["masked"] else None)


def run(state):
    kind = state["kind"]
    if kind == "masks":
        return state["pyramid"]()
    if kind == "step":
        state["graph"].replay()
        return state["outs"]
    if kind == "stack":
        outs, masks_ = state["net"].run(state["x"], state["mask"], keep_outputs=state["keep"], chain=state["chain"],
                                        compact=state["compact"])
        last = max(outs)
        return [outs[i] for i in sorted(outs) if i >= 0] if state["keep"] else outs[last]
    if kind == "grouped":
        return B.focused_gconv2d(state["desc"], state["groups"], state["x"], state["weights"], state["bias"],
                                 mask_in=state["mask"])
    return B.focused_conv2d(state["desc"], state["x"], state["weights"], state["bias"], mask_in=state["mask"])


# ---- what a pass cannot do without ---------------------------------------------

def _halved(v):
    return (v - 1) // 2 + 1


def _conv_work(n, h, w, c_in, c_out, k, stride, ho, wo, kept, groups, in_bytes, out_bytes, zero_fill=True):
    """Kept pixels read once, weights once, the output written once (all of it when it is zero-filled)."""
    m = n * ho * wo
    read = min(kept * n * h * w, kept * m * k * k) * c_in * in_bytes
    write = m * c_out * out_bytes * (1.0 if zero_fill else kept)
    return (read + write + c_out * k * k * (c_in // groups) * in_bytes,
            2.0 * kept * m * k * k * (c_in // groups) * c_out)


def _masks_work(n, h, w, levels, kept, packed=False):
    size = 1 / 8 if packed else 1
    bytes_ = n * h * w                       # the input mask, then per level its mask and its list
    for level in range(levels):
        bytes_ += n * h * w * (size + 4 * kept)
        h, w = _halved(h), _halved(w)
    return bytes_


def work(case):
    kind = case["kind"]
    kept = 1.0 - case["irrelevant"]
    n = case["n"]
    if kind == "masks":
        return {"bytes": _masks_work(n, case["h"], case["w"], case["levels"], kept, case["packed"]), "flops": 0}
    if kind == "step":
        h = case["side"]
        bytes_, flops = _masks_work(n, h, h, 4, kept), 0.0
        for c, _ in workloads.sweep_shapes():
            b, f = _conv_work(n, h, h, c, c, 3, 1, h, h, kept, 1, BYTES[case["dtype"]], max(2, BYTES[case["dtype"]]))
            bytes_, flops, h = bytes_ + b, flops + f, _halved(h)
        return {"bytes": bytes_, "flops": flops}
    in_bytes = BYTES[case["dtype"]]
    if kind in ("layer", "grouped"):
        if not case["masked"]:
            kept = 1.0
        h, w, k, s = case["h"], case["w"], case["k"], case["stride"]
        ho, wo = (h - 1 + 2 * (k // 2) - (k - 1)) // s + 1, (w - 1 + 2 * (k // 2) - (k - 1)) // s + 1
        out_bytes = 4 if case["out"] == "f32" else max(2, in_bytes)
        b, f = _conv_work(n, h, w, case["c_in"], case["c_out"], k, s, ho, wo, kept, case["groups"], in_bytes, out_bytes)
        return {"bytes": b + (n * h * w if case["masked"] else 0), "flops": f}
    # a stack: layer by layer, the feature maps between layers do not fit on the chip
    sizes = {-1: (case["h"], case["w"])}
    ops = NETWORKS[case["net"]][0]()
    bytes_, flops = float(n * case["h"] * case["w"]), 0.0
    for i, op in enumerate(ops):
        h, w = sizes[op.src]
        ho, wo = (h + 2 * op.pad - op.k) // op.stride + 1, (w + 2 * op.pad - op.k) // op.stride + 1
        sizes[i] = (ho, wo)
        if op.kind == "maxpool":
            bytes_ += kept * n * (h * w + ho * wo) * op.c_in * in_bytes
            continue
        fill = not case["chain"] or i == len(ops) - 1
        b, f = _conv_work(n, h, w, op.c_in, op.c_out, op.k, op.stride, ho, wo, kept,
                          op.c_in if op.kind == "dwconv" else 1, in_bytes, in_bytes, fill)
        bytes_, flops = bytes_ + b, flops + f
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "masks":
        return "exact"
    if kind == "stack":
        # one rounding per layer, carried through all of them
        return {"rel": {"bf16": 1e-2, "f16": 2e-3, "fp8": 3e-2}[case["dtype"]], "max": 0.5 if case["dtype"] == "fp8" else 0.1}
    if kind in ("layer", "grouped") and "f32" in (case["out"], case["dtype"]):
        return {"rel": 1e-5, "max": 1e-4}
    # sums in fp32, one rounding of the result: another order of summation moves a few of them by one place
    return {"rel": {"bf16": 2e-3, "f16": 3e-4, "fp8": 2e-3}[case["dtype"]], "max": 1e-2}
