"""Performance cases: forward passes of CNN partitions as a serving node runs them.

A node holds one or more partitions (contiguous layer ranges of a CNN) and runs
each on batches of 1 to 64 images or boundary feature maps.  A case is one such
pass through `Partition.run` (and `cast` where two partitions meet):

  model, begin, end   the architecture and the layer range [begin, end)
  dtype               storage type of activations and weights (f32, f16, bf16)
  batch               images per pass
  side                height and width of the model's input image; a range that
                      starts in the middle gets the feature map that follows
  mode                "graph": a captured graph over fixed buffers is replayed (a
                      server's steady state); "direct": the kernels are launched
                      on the caller's stream (buffers that change from call to
                      call); "static": direct launches with the library's fixed
                      scratch memory (callers that must not allocate)
  cut                 0, or a layer in (begin, end) where an fp32 range is split
                      into two partitions with the feature map quantised to fp16
                      in between, as it crosses from one pool to the next

`draw` spreads over the same ranges: any model, any valid range of up to twelve
layers, every storage type, any batch from 1 to 64 and images from 96 to 256
pixels a side, odd ones among them.
"""
import math

import torch

from paper_2507_18748_amd import Partition, cast
from workloads import zoo

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BN_EPS = 1e-5


def listed():
    def case(name, model, begin, end, dtype, batch, mode="graph", side=224, cut=0):
        return {"name": name, "model": model, "begin": begin, "end": end, "dtype": dtype,
                "batch": batch, "side": side, "mode": mode, "cut": cut}

    return [
        # whole-model serving at the largest batch: the benchmark's default
        case("resnet152_f16_b64", "resnet152", 0, 158, "f16", 64),
        # the same model for a single request, where every layer's latency counts
        case("resnet152_f16_b1", "resnet152", 0, 158, "f16", 1),
        # a planner's block in the middle of a deep network at an uneven batch
        case("resnet152_block_f16_b13", "resnet152", 28, 44, "f16", 13),
        # the last partition of a two-stage pipeline, at a pool's usual batch
        case("resnet50_layer4_head_bf16_b8", "resnet50", 44, 56, "bf16", 8),
        # a middle partition on odd feature maps (from 200-pixel images), buffers passed per call
        case("resnet50_layer3_bf16_b27", "resnet50", 25, 44, "bf16", 27, "direct", side=200),
        # the smallest call: pooling, classifier and softmax of one image
        case("resnet50_head_bf16_b1", "resnet50", 54, 56, "bf16", 1, "direct"),
        # the first fp32 partition at batch 1, launched per call
        case("resnet18_stem_layer1_f32_b1", "resnet18", 0, 6, "f32", 1, "direct"),
        # two fp32 partitions with the fp16 boundary between them
        case("resnet18_two_parts_f32_b16", "resnet18", 0, 16, "f32", 16, "direct", cut=6),
        # the convolutional part of VGG-16: the compute-heavy end of the range
        case("vgg16_features_f16_b16", "vgg16", 0, 18, "f16", 16),
        # its classifier at a small batch: 247 MB of weights, next to no arithmetic
        case("vgg16_classifier_f16_b4", "vgg16", 18, 21, "f16", 4, "static"),
        # depthwise-separable layers on large maps: bound by memory
        case("mobilenet_v2_early_bf16_b32", "mobilenet_v2", 0, 15, "bf16", 32),
        # and on small ones, at a small batch
        case("mobilenet_v2_late_f16_b5", "mobilenet_v2", 39, 54, "f16", 5),
    ]


def _model(name):
    return zoo.model(name)


def _shapes(m, side):
    """Output (c, h, w) of every layer; index -1 (the last entry) is the image."""
    out = []
    for L in m.layers:
        _, h, w = out[L.src] if L.src >= 0 else (m.in_c, side, side)
        if L.op in ("conv", "maxpool"):
            h = (h + 2 * L.pad - L.k) // L.stride + 1
            w = (w + 2 * L.pad - L.k) // L.stride + 1
        else:
            h = w = 1
        out.append((L.c_out, h, w))
    return out + [(m.in_c, side, side)]


def _in_shape(m, shapes, begin):
    return shapes[begin - 1] if begin > 0 else shapes[-1]


def _starts(m):
    """Boundaries p where every layer from p on reads only layer p - 1 or later."""
    n = len(m.layers)
    ok = []
    for p in range(n + 1):
        reads = [s for L in m.layers[p:] for s in (L.src, L.res_src) if s >= 0]
        image = any(L.src < 0 for L in m.layers[p:])
        ok.append(p == 0 or (not image and all(s >= p - 1 for s in reads)))
    return ok


def draw(rng):
    while True:
        name = rng.choice(("resnet18", "resnet50", "resnet152", "vgg16", "mobilenet_v2"))
        m = _model(name)
        n = len(m.layers)
        ok = [p for p, good in enumerate(_starts(m)) if good]
        begin = rng.choice(ok[:-1])
        ends = [p for p in ok if begin < p <= begin + 12]
        if not ends:
            continue
        end = rng.choice(ends)
        # VGG's classifier is defined for 224-pixel images only
        fixed = name == "vgg16" and end > 18
        side = 224 if fixed else rng.choice((224, rng.randint(96, 256)))
        case = {"model": name, "begin": begin, "end": end,
                "dtype": rng.choice(("f16", "f16", "bf16", "bf16", "f32")),
                "batch": int(round(2 ** rng.uniform(0, 6))), "side": side,
                "mode": rng.choice(("graph", "graph", "direct", "static")), "cut": 0}
        if case["dtype"] == "f32":
            # the library's fixed scratch is for small runs; fp32 goes out directly
            case["mode"] = rng.choice(("graph", "direct"))
            cuts = [p for p in ok if begin < p < end]
            if cuts and rng.random() < 0.5:
                case["mode"], case["cut"] = "direct", rng.choice(cuts)
        if case["mode"] == "static" and case["batch"] > 16:
            case["mode"] = "direct"
        w = work(case)
        # fp32 runs at a sixteenth of the 16-bit rate
        if w["flops"] * (16 if case["dtype"] == "f32" else 1) <= 1.2e12 and n >= end:
            return case


def _params(m, begin, end, dtype, g):
    """He-initialised weights (smaller in the classifier, 0.01, or 0.002 behind a
    whole network's larger features, so that the softmax does not saturate) and batch-norm statistics, representable in
    dtype; the last batch norm before each residual add has gamma 0.2, as it is
    small in trained networks (at 1 the activations of a deep one leave fp16)."""
    P = {}
    for i in range(begin, end):
        L = m.layers[i]
        if L.op not in ("conv", "fc", "fc_softmax"):
            continue
        shape = (L.c_out, L.c_in // L.groups, L.k, L.k) if L.op == "conv" else (L.c_out, L.c_in)
        fan_in = math.prod(shape[1:])
        std = math.sqrt(2.0 / fan_in)
        if L.op == "fc_softmax":
            std = 0.002 if begin == 0 else 0.01
        w = torch.randn(shape, generator=g, device="cuda") * std
        p = {"weight": w.to(TORCH[dtype]).float()}
        if L.bias:
            p["bias"] = torch.randn(L.c_out, generator=g, device="cuda") * 0.01
        if L.bn:
            p["bn_gamma"] = torch.full((L.c_out,), 0.2 if L.res_src >= 0 else 1.0, device="cuda")
            p["bn_beta"] = torch.zeros(L.c_out, device="cuda")
            p["bn_mean"] = torch.randn(L.c_out, generator=g, device="cuda") * 0.1
            p["bn_var"] = torch.rand(L.c_out, generator=g, device="cuda") + 0.5
        P[i] = p
    return P


def _inputs(case, seed):
    """Model, parameters and input (NHWC, in the storage type) from the seed alone."""
    m = _model(case["model"])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    c, h, w = _in_shape(m, _shapes(m, case["side"]), case["begin"])
    shape = (case["batch"], h, w, c)
    if case["begin"] == 0:  # normalised image
        mean = torch.tensor((0.485, 0.456, 0.406), device="cuda")
        std = torch.tensor((0.229, 0.224, 0.225), device="cuda")
        x = (torch.rand(shape, generator=g, device="cuda") - mean) / std
    else:  # boundary feature map, after an activation
        x = torch.randn(shape, generator=g, device="cuda").clamp_(min=0)
    P = _params(m, case["begin"], case["end"], case["dtype"], g)
    return m, P, x.to(TORCH[case["dtype"]]).contiguous()


def prepare(case, seed):
    m, P, x = _inputs(case, seed)
    host = {i: {k: v.cpu().numpy() for k, v in p.items()} for i, p in P.items()}
    del P
    shapes = _shapes(m, case["side"])
    ends = [case["begin"]] + ([case["cut"]] if case["cut"] else []) + [case["end"]]
    parts, bufs = [], [x]
    for b, e in zip(ends, ends[1:]):
        part = Partition(m.layers, host, (m.in_c, case["side"], case["side"]), b, e,
                         case["dtype"], max_batch=case["batch"], bn_eps=BN_EPS)
        parts.append(part)
        c, h, w = shapes[e - 1]
        dt = torch.float32 if m.layers[e - 1].op == "fc_softmax" else TORCH[case["dtype"]]
        bufs.append(torch.empty((case["batch"], h, w, c), dtype=dt, device="cuda"))
    state = {"parts": parts, "bufs": bufs, "batch": case["batch"], "mode": case["mode"]}
    if case["cut"]:
        state["wire"] = torch.empty(bufs[1].shape, dtype=torch.float16, device="cuda")
        state["recv"] = torch.empty_like(bufs[1])
    if case["mode"] == "graph":
        parts[0].capture(case["batch"], x.data_ptr(), bufs[1].data_ptr())
    return state


def run(state):
    parts, bufs, b = state["parts"], state["bufs"], state["batch"]
    stream = torch.cuda.current_stream().cuda_stream
    if state["mode"] == "static":
        parts[0].run_static_scratch(b, bufs[0].data_ptr(), bufs[1].data_ptr(), stream)
        return bufs[1]
    parts[0].run(b, bufs[0].data_ptr(), bufs[1].data_ptr(), stream)
    if "wire" not in state:
        return bufs[1]
    wire, recv = state["wire"], state["recv"]
    cast(bufs[1].data_ptr(), "f32", wire.data_ptr(), "f16", wire.numel(), stream)
    cast(wire.data_ptr(), "f16", recv.data_ptr(), "f32", wire.numel(), stream)
    parts[1].run(b, recv.data_ptr(), bufs[2].data_ptr(), stream)
    return {"boundary": wire, "out": bufs[2]}


def work(case):
    """Input, parameters and output once each (feature maps between the layers
    need not leave the chip), two operations per multiply-add."""
    m = _model(case["model"])
    shapes = _shapes(m, case["side"])
    size = 4 if case["dtype"] == "f32" else 2
    b = case["batch"]
    bytes_ = b * math.prod(_in_shape(m, shapes, case["begin"])) * size
    last = m.layers[case["end"] - 1]
    bytes_ += b * math.prod(shapes[case["end"] - 1]) * (4 if last.op == "fc_softmax" else size)
    if case["cut"]:  # the boundary map is written and read in fp16
        bytes_ += 2 * 2 * b * math.prod(shapes[case["cut"] - 1])
    flops = 0
    for i in range(case["begin"], case["end"]):
        L = m.layers[i]
        c, h, w = shapes[i]
        if L.op == "conv":
            k = (L.c_in // L.groups) * L.k * L.k
        elif L.op in ("fc", "fc_softmax"):
            k = L.c_in
        elif L.op == "maxpool":
            flops += b * c * h * w * L.k * L.k
            continue
        else:
            flops += b * math.prod(shapes[L.src])
            continue
        flops += 2 * b * c * h * w * k
        bytes_ += L.c_out * k * size + 8 * L.c_out
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times the error measured against 64-bit arithmetic (every
    stored feature map is rounded to the storage type on the way)."""
    if case["cut"]:  # a boundary value may round to either fp16 neighbour
        return {"rel": 1e-3, "max": 8e-3}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if case["dtype"] == "f16":
        whole = case["end"] - case["begin"] > 20  # roundings travel through many layers
        return {"rel": 5e-3, "max": 4e-2} if whole else {"rel": 2.5e-3, "max": 2e-2}
    return {"rel": 2.5e-2, "max": 0.15}


def _conv64(x, w, L):
    """x [N, C, H, W], w [Co, C / groups, k, k]: one matrix product per tap."""
    n, c, h, wd = x.shape
    ho, wo = (h + 2 * L.pad - L.k) // L.stride + 1, (wd + 2 * L.pad - L.k) // L.stride + 1
    x = torch.nn.functional.pad(x, (L.pad,) * 4)
    y = torch.zeros((n, L.c_out, ho, wo), dtype=torch.float64, device=x.device)
    for i in range(L.k):
        for j in range(L.k):
            s = x[:, :, i:i + (ho - 1) * L.stride + 1:L.stride,
                  j:j + (wo - 1) * L.stride + 1:L.stride]
            if L.groups > 1:
                y += s * w[:, 0, i, j].view(1, -1, 1, 1)
            else:
                s = s.permute(1, 0, 2, 3).reshape(c, -1)
                y += (w[:, :, i, j].contiguous() @ s).view(L.c_out, n, ho, wo).transpose(0, 1)
    return y


def exact(case, seed):
    m, P, x = _inputs(case, seed)
    begin, end = case["begin"], case["end"]
    last_use = {}
    for i in range(begin, end):
        for s in (m.layers[i].src, m.layers[i].res_src):
            last_use[s] = i
    act = {begin - 1: x.double().permute(0, 3, 1, 2)}
    wire = None
    for i in range(begin, end):
        L, p = m.layers[i], {k: v.double() for k, v in P.get(i, {}).items()}
        a = act[L.src]
        if L.op == "conv":
            y = _conv64(a, p["weight"], L)
            if "bias" in p:
                y += p["bias"].view(1, -1, 1, 1)
            if "bn_var" in p:
                s = p["bn_gamma"] / torch.sqrt(p["bn_var"] + BN_EPS)
                y = (y - p["bn_mean"].view(1, -1, 1, 1)) * s.view(1, -1, 1, 1) \
                    + p["bn_beta"].view(1, -1, 1, 1)
            if L.res_src >= 0:
                y = y + act[L.res_src]
        elif L.op == "maxpool":
            a = torch.nn.functional.pad(a, (L.pad,) * 4, value=-math.inf)
            y = a.unfold(2, L.k, L.stride).unfold(3, L.k, L.stride).amax((-1, -2))
        elif L.op == "gap":
            y = a.mean((2, 3), keepdim=True)
        else:
            y = (a.reshape(a.shape[0], -1) @ p["weight"].T + p["bias"])[:, :, None, None]
        if L.act != "none":
            y = y.clamp(min=0, max=6 if L.act == "relu6" else None)
        if L.op == "fc_softmax":
            y = torch.softmax(y, 1)
        act[i] = y
        for s in [s for s, u in last_use.items() if u == i and s in act]:
            del act[s]
        if case["cut"] and i == case["cut"] - 1:
            wire = y.permute(0, 2, 3, 1)
    out = act[end - 1].permute(0, 2, 3, 1).contiguous()
    if case["cut"]:
        return {"boundary": wire.contiguous(), "out": out}
    return out


if __name__ == "__main__":  # what is measured, in one line each
    for c in listed():
        w = work(c)
        print(f"{c['name']:32s} {w['bytes'] / 1e6:8.1f} MB {w['flops'] / 1e9:8.1f} GFLOP")
