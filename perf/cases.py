"""The work this library is measured on: int8 convolution layers as a user's program calls them through the binding.

listed()   the fixed cases, from one small layer (a call is all launch and host time) to a deep layer over a large batch
draw()     more layers of the same kinds, sizes spread over the ranges the listed ones stand for
prepare()  what the program holds before the call: tensors on the GPU and, where a serving program keeps them, rewritten
           weights and buffers
run()      one pass through the public entry points, its outputs whole
work()     bytes and operations the pass cannot do without (every input read once, every output written once)

Kinds of pass ("op"):
  conv      conv2d_int8 on raw NCHW / KCRS tensors: the one-shot call, everything rewritten within it
  pair      two one-shot calls, a 3x3 layer and a 1x1 layer on the same maps (each on an input of its own)
  serve     conv2d_int8_ex with weights rewritten once beforehand, workspace and output kept (a serving loop)
  chain     blocked inference chain: pack_layout, 3x3 layer with the activation in its epilogue, 1x1 layer on its blocked result
  nhwc      conv2d_int8_nhwc, a 3x3 layer and a 1x1 layer of an NHWC network
  dilated   a dilated 3x3 layer, by the batch route ("batch") or the address multiplier ("direct")
  rewrites  the individually callable layout rewrites around one layer (channel blocking, stencil unrolling, activation with
            the next layer's blocking, unpacking to NHWC)
"""
import math

import torch

from paper_2104_04731_amd import binding as conv


def _layer(name, op, N, C, H, W, K, R, S, stride, pad, dist="uniform", **more):
    return dict(name=name, op=op, N=N, C=C, H=H, W=W, K=K, R=R, S=S, stride=stride, pad=pad, dist=dist, **more)


def listed():
    return [
        # one small layer at batch 1: what a single call costs
        _layer("tiny 3x3 16ch n1", "conv", 1, 16, 14, 14, 16, 3, 3, 1, 1),
        # the headline step: a deep 3x3 layer and the 1x1 layer behind it at an online batch
        _layer("deep pair n8", "pair", 8, 256, 14, 14, 512, 3, 3, 1, 1, K2=128),
        # the three-channel stem of an image network, online batch
        _layer("stem 7x7 n4", "conv", 4, 3, 224, 224, 64, 7, 7, 2, 3),
        # the same stem over an offline batch
        _layer("stem 7x7 n512", "conv", 512, 3, 224, 224, 64, 7, 7, 2, 3),
        # the one-channel speech layer on spectrograms (clipped normal values)
        _layer("speech 20x5 n4", "conv", 4, 1, 161, 500, 32, 20, 5, 2, 0, "normal"),
        # channel counts that fill no block and a stride: a down-sampling layer at a medium batch
        _layer("ragged 72ch s2 n16", "conv", 16, 72, 56, 56, 96, 3, 3, 2, 1),
        # an early 3x3 layer in a serving loop: weights rewritten once, everything else per call
        _layer("serve 64ch n64", "serve", 64, 64, 56, 56, 64, 3, 3, 1, 1),
        # the deep layer over an offline batch: the matrix product decides
        _layer("serve deep n2048", "serve", 2048, 256, 14, 14, 512, 3, 3, 1, 1),
        # two layers that stay blocked between them, activation fused
        _layer("chain n32", "chain", 32, 256, 14, 14, 512, 3, 3, 1, 1, "normal", K2=128),
        # an NHWC block at a medium batch
        _layer("nhwc block n64", "nhwc", 64, 128, 28, 28, 128, 3, 3, 1, 1, K2=256),
        # a dilated layer (context module), the paper's route
        _layer("dilated d2 n64", "dilated", 64, 64, 28, 28, 64, 3, 3, 1, 2, dilation=2, route="batch"),
        # the rewrites on their own, large enough for memory to decide
        _layer("rewrites 64ch n256", "rewrites", 256, 64, 56, 56, 64, 3, 3, 1, 1),
    ]


# The largest listed layer bounds what a drawn one may cost.
MOST_OPS, MOST_BYTES = 4.0e11, 6.0e8


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, hi, case):
    """A batch size between 1 and `hi`, spread over its logarithm, within the bounds on a drawn case's cost."""
    one = work(dict(case, N=1))
    top = min(hi, int(MOST_OPS / max(one["flops"], 1.0)), int(MOST_BYTES / one["bytes"]))
    return _log_int(rng, 1, max(1, top))


def _many_channels(rng):
    """A layer of the body of an image network: C grows as the maps shrink, sometimes not a multiple of any block."""
    H = rng.choice([7, 14, 28, 56]) if rng.random() < 0.6 else _log_int(rng, 7, 60)
    C = rng.choice([32, 64, 128, 256, 512]) if rng.random() < 0.6 else _log_int(rng, 16, 512)
    K = rng.choice([32, 64, 128, 256, 512]) if rng.random() < 0.6 else _log_int(rng, 16, 512)
    return H, C, K


def draw(rng):
    kind = rng.choice(["body", "body", "pointwise", "stem", "speech", "pair", "serve", "serve", "chain", "nhwc", "dilated", "rewrites"])
    dist = rng.choice(["uniform", "normal"])
    H, C, K = _many_channels(rng)
    if kind == "body":
        R = rng.choice([3, 3, 3, 5])
        c = dict(op="conv", N=1, C=C, H=H, W=H + rng.choice([0, 0, 0, 1, 5]), K=K, R=R, S=R, stride=rng.choice([1, 1, 2]), pad=R // 2)
    elif kind == "pointwise":
        c = dict(op="conv", N=1, C=C, H=H, W=H, K=K, R=1, S=1, stride=rng.choice([1, 1, 1, 2]), pad=0)
    elif kind == "stem":
        R = rng.choice([3, 5, 7])
        c = dict(op="conv", N=1, C=rng.choice([1, 3, 3, 4]), H=_log_int(rng, 96, 256), W=_log_int(rng, 96, 256), K=rng.choice([16, 24, 32, 64]),
                 R=R, S=R, stride=rng.choice([1, 2, 2]), pad=R // 2)
    elif kind == "speech":
        c = dict(op="conv", N=1, C=1, H=rng.choice([151, 161]), W=_log_int(rng, 200, 720), K=rng.choice([32, 64]), R=rng.choice([5, 20]), S=5,
                 stride=2, pad=rng.choice([0, 1]))
    elif kind == "pair":
        c = dict(op="pair", N=1, C=C, H=H, W=H, K=K, R=3, S=3, stride=1, pad=1, K2=_log_int(rng, 32, 256))
    elif kind == "serve":
        c = dict(op="serve", N=1, C=C, H=H, W=H, K=K, R=3, S=3, stride=rng.choice([1, 1, 2]), pad=1)
    elif kind == "chain":
        c = dict(op="chain", N=1, C=C, H=H, W=H, K=K, R=3, S=3, stride=1, pad=1, K2=_log_int(rng, 32, 256))
    elif kind == "nhwc":
        c = dict(op="nhwc", N=1, C=C, H=H, W=H, K=K, R=3, S=3, stride=1, pad=1, K2=_log_int(rng, 32, 512))
    elif kind == "dilated":
        d = rng.choice([2, 2, 3, 4])
        c = dict(op="dilated", N=1, C=C, H=max(H, 14), W=max(H, 14), K=K, R=3, S=3, stride=1, pad=d, dilation=d, route=rng.choice(["batch", "direct"]))
    else:
        c = dict(op="rewrites", N=1, C=C, H=H, W=H + rng.choice([0, 0, 1]), K=K, R=3, S=3, stride=rng.choice([1, 1, 2]), pad=1)
    c["dist"] = dist
    c["N"] = _batch(rng, 1024, c)
    return c


def _dims(c):
    return (c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["S"], c["stride"], c["pad"])


def _pixels(c):
    d = c.get("dilation", 1)
    P = (c["H"] + 2 * c["pad"] - d * (c["R"] - 1) - 1) // c["stride"] + 1
    Q = (c["W"] + 2 * c["pad"] - d * (c["S"] - 1) - 1) // c["stride"] + 1
    return P, Q


def _int8(gen, shape, dist):
    """Quantised activations and weights: uniform over the type, or a normal distribution of deviation 32 clipped to it."""
    if dist == "uniform":
        return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=gen)
    return torch.randn(shape, device="cuda", generator=gen).mul_(32.0).round_().clamp_(-128, 127).to(torch.int8)


def _second(c):
    """The 1x1 layer behind a 3x3 layer, on that layer's result."""
    P, Q = _pixels(c)
    return dict(N=c["N"], C=c["K"], H=P, W=Q, K=c["K2"], R=1, S=1, stride=1, pad=0)


def prepare(case, seed):
    c = case
    op = c["op"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dims = _dims(c)
    N, C, H, W, K, R, S, stride, pad = dims
    P, Q = _pixels(c)
    s = dict(case=c, dims=dims)
    s["x"] = _int8(gen, (N, H, W, C) if op == "nhwc" else (N, C, H, W), c["dist"])
    s["w"] = _int8(gen, (K, C, R, S), c["dist"])
    if op in ("pair", "nhwc", "chain"):
        s["w2"] = _int8(gen, (c["K2"], K, 1, 1), c["dist"])
    if op == "pair":
        s["x2"] = _int8(gen, (N, K, P, Q), c["dist"])
    elif op == "nhwc":
        s["x2"] = _int8(gen, (N, P, Q, K), c["dist"])
    elif op == "serve":
        # a serving program rewrites its weights when it loads them and keeps workspace and output
        lay, cb, _ = conv.select_layout(dims)
        if lay == conv.LAYOUT_IMAGE_PACK:  # its weights are not a single rewrite
            lay, cb = conv.LAYOUT_PACKED, 64 if C > 32 else 32 if C > 16 else 16
        s["layout"], s["cb"] = lay, cb
        s["wq"] = conv.pack_weights(s["w"], lay, cb)
        need = conv.conv2d_int8_workspace_bytes(dims, lay, cb, True)
        s["ws"] = torch.empty(max(need, 256), dtype=torch.int8, device="cuda")
        s["out"] = torch.empty((N, K, P, Q), dtype=torch.int32, device="cuda")
    elif op == "chain":
        d2 = _second(c)
        s["dims2"] = _dims(d2)
        s["cb"], s["cb2"] = 64 if C > 32 else 32 if C > 16 else 16, 64 if K > 32 else 32 if K > 16 else 16
        s["wq"] = conv.pack_weights(s["w"], conv.LAYOUT_PACKED, s["cb"])
        s["wq2"] = conv.pack_weights(s["w2"], conv.LAYOUT_PACKED, s["cb2"])
        s["xq"] = torch.empty(conv.pack_layout_bytes(N, C, H, W, s["cb"], pad), dtype=torch.int8, device="cuda")
        s["mid"] = torch.empty((N, -(-K // s["cb2"]), P, Q, s["cb2"]), dtype=torch.int8, device="cuda")
        s["out"] = torch.empty((N, c["K2"], P, Q), dtype=torch.int32, device="cuda")
        # the shift that brings accumulators of this depth back to int8 range
        s["shift"] = max(1, int(round(math.log2(math.sqrt(C * R * S) * 32.0))))
    elif op == "rewrites":
        # int32 results of a layer of this depth
        s["acc"] = torch.randn((N, K, P, Q), device="cuda", generator=gen).mul_(1024.0 * math.sqrt(C * R * S)).to(torch.int32)
        s["shift"] = max(1, int(round(math.log2(math.sqrt(C * R * S) * 32.0))))
        s["cb"], s["cb2"] = 64 if C > 32 else 32 if C > 16 else 16, 64 if K > 32 else 32 if K > 16 else 16
    return s


def run(state):
    s, c = state, state["case"]
    op = c["op"]
    if op == "conv":
        return conv.conv2d_int8(s["x"], s["w"], c["stride"], c["pad"])
    if op == "pair":
        return [conv.conv2d_int8(s["x"], s["w"], c["stride"], c["pad"]), conv.conv2d_int8(s["x2"], s["w2"], 1, 0)]
    if op == "serve":
        return conv.conv2d_int8_ex(s["dims"], s["layout"], s["cb"], s["x"], s["wq"], s["out"], s["ws"], wt_is_packed=True)
    if op == "chain":
        conv.pack_layout(s["x"], s["cb"], c["pad"], out=s["xq"])
        conv.conv2d_int8_packed_requant(s["dims"], conv.LAYOUT_PACKED, s["cb"], s["xq"], s["wq"], s["cb2"], 0, s["shift"], True, out=s["mid"])
        conv.conv2d_int8_packed(s["dims2"], conv.LAYOUT_PACKED, s["cb2"], s["mid"], s["wq2"], s["out"])
        return [s["mid"], s["out"]]
    if op == "nhwc":
        return [conv.conv2d_int8_nhwc(s["x"], s["w"], c["stride"], c["pad"]), conv.conv2d_int8_nhwc(s["x2"], s["w2"], 1, 0)]
    if op == "dilated":
        route = conv.conv2d_int8_dilated if c["route"] == "batch" else conv.conv2d_int8_dilated_direct
        return route(s["dims"], c["dilation"], s["x"], s["w"])
    return [conv.pack_layout(s["x"], s["cb"], c["pad"]), conv.im2col_int8(s["x"], c["R"], c["S"], c["stride"], c["pad"]),
            conv.requant_pack_layout(s["acc"], s["cb2"], c["pad"], s["shift"], True), conv.unpack_nhwc_int32(s["acc"])]


def _conv_work(c):
    N, C, H, W, K, R, S, stride, pad = _dims(c)
    P, Q = _pixels(c)
    return N * C * H * W, K * C * R * S, N * K * P * Q, 2 * N * K * P * Q * C * R * S


def work(case):
    c = case
    op = c["op"]
    x, w, o, ops = _conv_work(c)
    if op == "rewrites":
        N, C, H, W, K, R, S, stride, pad = _dims(c)
        P, Q = _pixels(c)
        cb, cb2 = 64 if C > 32 else 32 if C > 16 else 16, 64 if K > 32 else 32 if K > 16 else 16
        packed = N * -(-C // cb) * cb * (H + 2 * pad) * (W + 2 * pad)
        unrolled = N * P * Q * (-(-C * R * S // 64) * 64)
        blocked = N * -(-K // cb2) * cb2 * (P + 2 * pad) * (Q + 2 * pad)
        return {"bytes": (x + packed) + (x + unrolled) + (4 * o + blocked) + (4 * o + 4 * o), "flops": 0}
    total = {"bytes": x + w + 4 * o, "flops": ops}
    if op in ("pair", "nhwc", "chain"):
        x2, w2, o2, ops2 = _conv_work(_second(c))
        total["flops"] += ops2
        if op == "chain":  # the layer between is int8, stored once and read once
            total["bytes"] = x + w + 2 * x2 + w2 + 4 * o2
        else:
            total["bytes"] += x2 + w2 + 4 * o2
    return total


def tolerance(case):
    # integer arithmetic without overflow: every summation order gives the same 32-bit words
    return "exact"
