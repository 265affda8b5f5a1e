"""The workloads whose speed is tracked, through the library's public entry points.

Each case is a plain dict.  ``prepare`` builds what a program holds before the
call (inputs, weights, packed filters, workspaces, a captured stack), ``run``
is one pass, ``exact`` the same result in 64 bits from plain torch.

Kinds of case:
  packed   one fp32/bf16 conv with filters packed once (PackedFilters.forward)
  layer    one conv layer planned as a Stack and replayed as a graph
  ws       one conv call with a caller workspace (conv2d_fwd_ws)
  cl       one bf16 channel-last conv (conv2d_fwd_cl), optionally with a join
  dw       one depthwise conv (dwconv2d_fwd)
  net      a whole network pass (Stack replay), returning the feature map of every stage
  scan, argsort, nms   the vision operators
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1907_02154_amd import detections, miconv, networks, vision

BF16, F32 = "bf16", "f32"


# ------------------------------------------------------------------ the cases

def _conv(name, kind, dtype, N, C, H, W, K, R, stride=1, pad=None, groups=1, relu=True, res=False):
    return {"name": name, "kind": kind, "dtype": dtype, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R,
            "stride": stride, "pad": R // 2 if pad is None else pad, "groups": groups, "relu": relu, "res": res}


def listed():
    return [
        # A single small layer called on its own at batch 1: launch and host latency.
        _conv("conv3x3_b1_f32", "packed", F32, 1, 64, 56, 56, 64, 3),
        # Batch-1 fp32 classification, the latency setting: 53 convs, max-pool, joins.
        {"name": "resnet50_b1_f32", "kind": "net", "net": "resnet50", "layout": "f32", "N": 1},
        # A VGG-16 3x3 layer at batch 8 in fp32: compute-bound, planned once and replayed.
        _conv("vgg3x3_b8_f32", "layer", F32, 8, 256, 56, 56, 256, 3),
        # Odd extents, a filter count that fills no tile, stride 2, a small batch.
        _conv("ragged_s2_b5_f32", "ws", F32, 5, 100, 55, 57, 120, 3, stride=2),
        # bf16 weights and activations in NCHW with an fp32 result, single calls at batch 64.
        _conv("conv3x3_b64_bf16", "ws", BF16, 64, 256, 14, 14, 256, 3),
        # The layers of a batch-64 channel-last network: a 3x3, and a wide 1x1 with the shortcut join.
        _conv("conv3x3_b64_cl", "cl", BF16, 64, 128, 28, 28, 128, 3),
        _conv("join1x1_b64_cl", "cl", BF16, 64, 64, 56, 56, 256, 1, res=True),
        # Batch-64 classification in bf16, activations channel-last between layers.
        {"name": "resnet50_b64_bf16_cl", "kind": "net", "net": "resnet50", "layout": "bf16_cl", "N": 64},
        # A MobileNet depthwise layer at a serving batch: bandwidth.
        {"name": "dw3x3_b64_f32", "kind": "dw", "N": 64, "C": 128, "H": 56, "W": 56, "stride": 1, "relu": True},
        # One long prefix sum: bandwidth.
        {"name": "scan_64M", "kind": "scan", "rows": 1, "n": 1 << 26, "exclusive": False},
        # Four million keys in segments of about a thousand.
        {"name": "argsort_4M", "kind": "argsort", "n": 1 << 22, "segments": 4096, "descending": True, "ties": False},
        # The detections of one image of an SSD-style detector: launch latency.
        {"name": "nms_b1", "kind": "nms", "N": 1, "rows": 24564, "topk": 400, "overlap": 0.45, "valid": 0.01,
         "force": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_conv(rng, kind, dtype):
    while True:
        R = rng.choice((1, 1, 3, 3, 3))
        N = _log(rng, 1, 64)
        H = _log(rng, 7, 112)
        W = H if rng.random() < 0.6 else max(7, H + rng.randint(-3, 3))
        stride = 2 if rng.random() < 0.2 else 1
        if kind == "cl":
            C, K = 64 * rng.choice((1, 2, 3, 4, 6, 8)), 8 * _log(rng, 6, 128)
        elif rng.random() < 0.6:
            C, K = 32 * rng.choice((1, 2, 3, 4, 6, 8, 16)), 32 * rng.choice((1, 2, 4, 6, 8, 16))
        else:
            C, K = _log(rng, 3, 400), _log(rng, 16, 500)
        c = _conv("", kind, dtype, N, C, H, W, K, R, stride, relu=rng.random() < 0.8,
                  res=kind in ("cl", "layer") and rng.random() < 0.3)
        del c["name"]
        w = work(c)
        if 2e7 < w["flops"] < 4e10 and w["bytes"] < 4e8:
            return c


def draw(rng):
    kind = rng.choice(("packed", "layer", "layer", "ws", "ws", "bf16", "bf16", "cl", "cl", "cl", "dw", "net",
                       "scan", "argsort", "nms"))
    if kind in ("packed", "layer"):
        return _draw_conv(rng, kind, F32)
    if kind == "ws":
        return _draw_conv(rng, "ws", F32)
    if kind == "bf16":
        return _draw_conv(rng, rng.choice(("ws", "layer")), BF16)
    if kind == "cl":
        return _draw_conv(rng, "cl", BF16)
    if kind == "dw":
        H = rng.choice((7, 14, 28, 56, 112, rng.randint(7, 112)))
        C = 16 * _log(rng, 2, 64)
        return {"kind": "dw", "N": max(1, min(_log(rng, 1, 128), int(4e7 / (C * H * H)))), "C": C, "H": H, "W": H,
                "stride": rng.choice((1, 1, 2)), "relu": rng.random() < 0.8}
    if kind == "net":
        net, layout, top = rng.choice((("resnet50", "f32", 4), ("mobilenet", "f32", 16), ("resnet50", "bf16_cl", 48)))
        return {"kind": "net", "net": net, "layout": layout, "N": _log(rng, 1, top)}
    if kind == "scan":
        total = _log(rng, 1 << 14, 1 << 26)
        rows = 1 if rng.random() < 0.5 else _log(rng, 1, 256)
        return {"kind": "scan", "rows": rows, "n": max(1, total // rows), "exclusive": rng.random() < 0.5}
    if kind == "argsort":
        n = _log(rng, 1 << 13, 1 << 22)
        return {"kind": "argsort", "n": n, "segments": min(n, _log(rng, 1, 8192)), "descending": rng.random() < 0.7,
                "ties": rng.random() < 0.3}
    rows = _log(rng, 1000, 30000)
    return {"kind": "nms", "N": _log(rng, 1, 32), "rows": rows, "topk": rng.choice((100, 200, 400, 1000)),
            "overlap": rng.choice((0.45, 0.5, 0.6)), "valid": 0.01, "force": rng.random() < 0.2}


# ------------------------------------------------------------- inputs, tensors

class _Rand:
    """Seeded device tensors with the distributions of the evaluated networks."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device="cuda")

    def normal(self, std, *shape):
        return torch.randn(shape, generator=self.g, device="cuda") * std


def _out(c):
    return ((c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1)


def _conv_tensors(c, seed):
    """x (NCHW, or NHWC for cl), He-normal w, bias N(0, 0.01), res like y; as the case stores them."""
    r = _Rand(seed)
    P, Q = _out(c)
    dt = torch.bfloat16 if c["dtype"] == BF16 else torch.float32
    cl = c["kind"] == "cl"
    cg = c["C"] // c["groups"]
    xs = (c["N"], c["H"], c["W"], c["C"]) if cl else (c["N"], c["C"], c["H"], c["W"])
    x = r.uniform(*xs).to(dt)
    w = r.normal(math.sqrt(2.0 / (cg * c["R"] * c["R"])), c["K"], cg, c["R"], c["R"]).to(dt)
    b = r.normal(0.01, c["K"])
    res = None
    if c["res"]:
        res = r.uniform(*((c["N"], P, Q, c["K"]) if cl else (c["N"], c["K"], P, Q)))
        res = res.to(torch.bfloat16) if cl else res
    return x, w, b, res


def _resnet50(N):
    """(name, source, K, R, stride, pad, relu, shortcut) of every conv; name "pool" is the 3x3/2 max-pool."""
    yield "stem", "input", 64, 7, 2, 3, True, None
    yield "pool", "stem", 0, 3, 2, 1, False, None
    prev = "pool"
    for s, (blocks, width) in enumerate(((3, 64), (4, 128), (6, 256), (3, 512)), start=2):
        for b in range(blocks):
            p, st, short = f"s{s}b{b}", 2 if b == 0 and s > 2 else 1, prev
            if b == 0:
                short = p + "proj"
                yield short, prev, 4 * width, 1, st, 0, False, None
            yield p + "c1", prev, width, 1, st, 0, True, None
            yield p + "c2", p + "c1", width, 3, 1, 1, True, None
            yield p + "c3", p + "c2", 4 * width, 1, 1, 0, True, short
            prev = p + "c3"


def _mobilenet(N):
    """The same for MobileNet-v1; K = -1 marks a depthwise conv."""
    yield "stem", "input", 32, 3, 2, 1, True, None
    prev = "stem"
    ks = (64, 128, 128, 256, 256, 512, 512, 512, 512, 512, 512, 1024, 1024)
    sts = (1, 2, 1, 2, 1, 2, 1, 1, 1, 1, 1, 2, 1)
    for i, (k, st) in enumerate(zip(ks, sts), start=1):
        yield f"dw{i}", prev, -1, 3, st, 1, True, None
        yield f"pw{i}", f"dw{i}", k, 1, 1, 0, True, None
        prev = f"pw{i}"


_NETS = {"resnet50": _resnet50, "mobilenet": _mobilenet}
# The feature maps that detectors and classifiers take from the pass: the last of every extent.
_STAGES = {"resnet50": ("s2b2c3", "s3b3c3", "s4b5c3", "s5b2c3"), "mobilenet": ("pw3", "pw5", "pw11", "pw13")}


def _net_tensors(c, seed):
    r = _Rand(seed)
    dt = torch.bfloat16 if c["layout"] == "bf16_cl" else torch.float32
    chans, params = {"input": 3}, {}
    for name, src, K, R, *_ in _NETS[c["net"]](c["N"]):
        C = chans[src]
        chans[name] = K if K > 0 else C
        if name == "pool":
            continue
        cg, k = (1, C) if K < 0 else (C, K)
        params[name] = (r.normal(math.sqrt(2.0 / (cg * R * R)), k, cg, R, R).to(dt), r.normal(0.01, k))
    return r.uniform(c["N"], 3, 224, 224).to(dt), params


# ------------------------------------------------------------------- the passes

def prepare(case, seed):
    c = case
    k = c["kind"]
    if k in ("packed", "layer", "ws"):
        x, w, b, res = _conv_tensors(c, seed)
        P, Q = _out(c)
        y = torch.empty((c["N"], c["K"], P, Q), device="cuda")
        s = {"c": c, "x": x, "w": w, "b": b, "y": y}
        if k == "packed":
            s["f"] = miconv.PackedFilters(w, tuple(x.shape), c["stride"], c["pad"], c["groups"])
        elif k == "ws":
            s["ws"] = miconv.workspace(miconv.conv2d_workspace_bytes(
                c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["R"], c["stride"], c["pad"], c["groups"], c["dtype"]))
        else:
            op = miconv.OP_CONV_BF16 if c["dtype"] == BF16 else miconv.OP_CONV_F32
            s["stack"] = miconv.Stack([(op, x, w, b, y, c["stride"], c["pad"], c["groups"], c["relu"], res)])
            s["stack"].capture(1, False)
        return s
    if k == "cl":
        x, w, b, res = _conv_tensors(c, seed)
        P, Q = _out(c)
        y = torch.empty((c["N"], P, Q, c["K"]), device="cuda", dtype=torch.bfloat16)
        ws = miconv.workspace(miconv.conv2d_cl_workspace_bytes(
            c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["R"], c["stride"], c["pad"], c["groups"]))
        return {"c": c, "x": x, "w": w, "b": b, "res": res, "y": y, "ws": ws}
    if k == "dw":
        r = _Rand(seed)
        P, Q = ((e - 1) // c["stride"] + 1 for e in (c["H"], c["W"]))
        return {"c": c, "x": r.uniform(c["N"], c["C"], c["H"], c["W"]), "w": r.normal(math.sqrt(2 / 9), c["C"], 1, 3, 3),
                "b": r.normal(0.01, c["C"]), "y": torch.empty((c["N"], c["C"], P, Q), device="cuda")}
    if k == "net":
        x, params = _net_tensors(c, seed)
        if c["net"] == "resnet50":
            graph = networks.resnet50_graph(5 if c["layout"] == "bf16_cl" else 2, c["N"])
        else:
            graph = networks.mobilenet_graph(c["N"])
        ops, outs = networks.build_stack(graph, x, params, c["layout"])
        stack = miconv.Stack(ops)
        stack.capture(1, False)
        return {"c": c, "stack": stack, "y": [outs[n] for n in _STAGES[c["net"]]]}
    if k == "scan":
        r = _Rand(seed)
        x = torch.randint(-1000, 1000, (c["rows"], c["n"]), generator=r.g, device="cuda", dtype=torch.int32)
        return {"c": c, "x": x, "y": torch.empty_like(x),
                "ws": miconv.workspace(vision.scan_workspace_bytes(c["rows"], c["n"]))}
    if k == "argsort":
        keys, off = _argsort_inputs(c, seed)
        return {"c": c, "x": keys, "off": off, "y": torch.empty(c["n"], device="cuda", dtype=torch.int32),
                "ws": miconv.workspace(vision.argsort_workspace_bytes(c["n"], c["segments"]))}
    x = torch.from_numpy(detections.detection_rows(c["N"], c["rows"], seed=seed)).cuda()
    return {"c": c, "x": x, "y": torch.empty_like(x),
            "ws": miconv.workspace(vision.box_nms_workspace_bytes(c["N"], c["rows"], 6, c["topk"]))}


def run(s):
    c = s["c"]
    k = c["kind"]
    if k == "packed":
        return s["f"].forward(s["x"], s["b"], s["y"], c["relu"])
    if k in ("layer", "net"):
        s["stack"].replay()
        return s["y"]
    if k == "ws":
        return miconv.conv2d_fwd_ws(s["x"], s["w"], s["b"], s["y"], c["stride"], c["pad"], c["groups"], c["relu"],
                                    ws=s["ws"])
    if k == "cl":
        return miconv.conv2d_fwd_cl(s["x"], s["w"], s["b"], s["y"], c["stride"], c["pad"], c["groups"], c["relu"],
                                    res=s["res"], ws=s["ws"])
    if k == "dw":
        return miconv.dwconv2d_fwd(s["x"], s["w"], s["b"], s["y"], c["stride"], 1, c["relu"])
    if k == "scan":
        return vision.scan_i32(s["x"], s["y"], exclusive=c["exclusive"], ws=s["ws"])
    if k == "argsort":
        return vision.segmented_argsort(s["x"], s["off"], c["descending"], out=s["y"], ws=s["ws"])
    return vision.box_nms(s["x"], c["overlap"], c["valid"], c["topk"], force_suppress=c["force"], out=s["y"], ws=s["ws"])


def _argsort_inputs(c, seed):
    r = _Rand(seed)
    if c["ties"]:
        keys = torch.randint(-8, 8, (c["n"],), generator=r.g, device="cuda").float()
    else:
        keys = r.normal(1.0, c["n"])
    return keys, torch.from_numpy(detections.segment_offsets(c["segments"], c["n"], seed)).cuda()


# ------------------------------------------------- work, tolerances, 64-bit result

def work(case):
    c = case
    k = c["kind"]
    if k == "scan":
        n = c["rows"] * c["n"]
        return {"bytes": 8 * n, "flops": n}
    if k == "argsort":
        return {"bytes": 8 * c["n"] + 4 * (c["segments"] + 1), "flops": 0}
    if k == "nms":
        return {"bytes": 2 * 24 * c["N"] * c["rows"], "flops": 0}
    if k == "net":
        # weights and biases, the image, the stages' feature maps
        ext, total, wbytes, maps = {"input": (224, 3)}, 0, 0, 0
        eb = 2 if c["layout"] == "bf16_cl" else 4
        for name, src, K, R, st, pad, _, _ in _NETS[c["net"]](c["N"]):
            e, C = ext[src]
            p = (e + 2 * pad - R) // st + 1
            ext[name] = (p, K if K > 0 else C)
            if name != "pool":
                cg = 1 if K < 0 else C
                total += 2 * c["N"] * ext[name][1] * p * p * cg * R * R
                wbytes += ext[name][1] * (cg * R * R * eb + 4)
            if name in _STAGES[c["net"]]:
                maps += c["N"] * ext[name][1] * p * p
        return {"bytes": wbytes + eb * (c["N"] * 3 * 224 * 224 + maps), "flops": total}
    if k == "dw":
        P, Q = ((e - 1) // c["stride"] + 1 for e in (c["H"], c["W"]))
        return {"bytes": 4 * (c["N"] * c["C"] * (c["H"] * c["W"] + P * Q) + 10 * c["C"]),
                "flops": 18 * c["N"] * c["C"] * P * Q}
    P, Q = _out(c)
    eb = 2 if c["dtype"] == BF16 else 4
    yb = 2 if k == "cl" else 4
    cg = c["C"] // c["groups"]
    ny = c["N"] * c["K"] * P * Q
    return {"bytes": eb * (c["N"] * c["C"] * c["H"] * c["W"] + c["K"] * cg * c["R"] ** 2) + 4 * c["K"]
            + yb * ny * (2 if c["res"] else 1),
            "flops": 2 * ny * cg * c["R"] ** 2}


def tolerance(case):
    """Relative 2-norm error: about four times what each path shows against the 64-bit result."""
    k = case["kind"]
    if k in ("scan", "argsort", "nms"):
        return "exact"
    if k == "net":
        return {"rel": 3e-2} if case["layout"] == "bf16_cl" else {"rel": 2e-6}
    if k == "cl":
        return {"rel": 7e-3}       # one rounding to bf16
    return {"rel": 2e-6}           # 32-bit sums of exactly representable inputs


def _conv64(x, w, b, stride, pad, relu, res=None):
    """conv2d in float64, NCHW, one matrix product per tap (one multiply per tap if depthwise)."""
    N, C, H, W = x.shape
    K, cg, R, S = w.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    y = torch.zeros((N, K, P, Q), dtype=torch.float64, device=x.device)
    for r in range(R):
        for s in range(S):
            t = xp[:, :, r:r + (P - 1) * stride + 1:stride, s:s + (Q - 1) * stride + 1:stride]
            if cg == 1 and K == C:
                y += t * w[:, 0, r, s].view(1, K, 1, 1)
            else:
                t = t.permute(1, 0, 2, 3).reshape(C, N * P * Q)
                y += torch.mm(w[:, :, r, s].contiguous(), t).view(K, N, P, Q).permute(1, 0, 2, 3)
    y += b.view(1, K, 1, 1)
    if res is not None:
        y += res
    return y.clamp_(min=0) if relu else y


def exact(case, seed):
    c = case
    k = c["kind"]
    if k == "nms":
        return None                # rows copied or -1, decided by fp32 comparisons
    if k == "scan":
        r = _Rand(seed)
        x = torch.randint(-1000, 1000, (c["rows"], c["n"]), generator=r.g, device="cuda", dtype=torch.int32)
        y = torch.cumsum(x, 1, dtype=torch.int64)
        return ((y - x) if c["exclusive"] else y).to(torch.int32)
    if k == "argsort":
        keys, off = _argsort_inputs(c, seed)
        kn, o = keys.cpu().numpy().astype(np.float64), off.cpu().numpy()
        seg = np.repeat(np.arange(c["segments"]), np.diff(o))
        order = np.lexsort((-kn if c["descending"] else kn, seg))    # stable
        return torch.from_numpy((order - o[:-1][seg]).astype(np.int32))
    if k == "dw":
        s = prepare(c, seed)
        return _conv64(s["x"].double(), s["w"].double(), s["b"].double(), c["stride"], 1, c["relu"])
    if k == "net":
        x, params = _net_tensors(c, seed)
        outs = {"input": x.double()}
        for name, src, _, R, st, pad, relu, short in _NETS[c["net"]](c["N"]):
            if name == "pool":
                outs[name] = torch.nn.functional.max_pool2d(outs[src], R, st, pad)
            else:
                w, b = params[name]
                outs[name] = _conv64(outs[src], w.double(), b.double(), st, pad, relu, outs[short] if short else None)
        ys = [outs[n] for n in _STAGES[c["net"]]]
        return [y.permute(0, 2, 3, 1).contiguous() for y in ys] if c["layout"] == "bf16_cl" else ys
    x, w, b, res = _conv_tensors(c, seed)
    res = None if res is None else res.double()
    x = x.double()
    if k == "cl":
        x, res = x.permute(0, 3, 1, 2), None if res is None else res.permute(0, 3, 1, 2)
    y = _conv64(x, w.double(), b.double(), c["stride"], c["pad"], c["relu"], res)
    return y.permute(0, 2, 3, 1).contiguous() if k == "cl" else y
