"""Performance cases of the elastic-kernel framework: the work its users have it do, through the
public entry points (paper_2307_04339_amd.ops, .models, .runtime).

A case is one layer, one block of layers that a network repeats, or one whole request.  Listed sizes
are those of the framework's own workloads (the single fp32 convolution, ResNet-18 at batch 1, VGG-16
at batch 8, MobileNetV2 at batch 16, the BERT-shaped encoder) plus generic odd and larger ones;
draw() spreads over the ranges those stand for.  Every activation stays in the buffers a program
keeps, and run() returns all of them.

exact() evaluates the same layers in float64 with plain torch, never rounding between layers.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2307_04339_amd import models, ops
from paper_2307_04339_amd.runtime import Coordinator

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one small fp32 convolution: the latency of a single call
        dict(name="conv_f32_56", kind="conv", dtype="f32", n=1, h=56, w=56, c=64, k=64, ks=3, stride=1, act="relu",
             bn=False, bias=True, residual=False, shards=1, block=256),
        # one residual block of ResNet-18's third stage at batch 1: few tiles, long K
        dict(name="resnet_block_b1", kind="basic", dtype="f16", n=1, h=14, c=256, k=256, stride=1),
        # a strided layer whose sizes no tile divides and whose channels are no whole chunk
        dict(name="conv_ragged", kind="conv", dtype="bf16", n=5, h=75, w=53, c=72, k=120, ks=3, stride=2, act="relu6",
             bn=True, bias=False, residual=False, shards=1, block=256),
        # best-effort work: a VGG-16 convolution issued as four elastic shards
        dict(name="conv_shards", kind="conv", dtype="f16", n=8, h=56, w=56, c=256, k=256, ks=3, stride=1, act="relu",
             bn=False, bias=True, residual=False, shards=4, block=256),
        # VGG-16 at batch 8, first stage: the image (3 channels stored as 8), large pixels, few channels
        dict(name="vgg_stage1_b8", kind="stage", dtype="f16", n=8, h=224, c=8, k=64, convs=2),
        # second stage: large pixels, 128 channels
        dict(name="vgg_stage2_b8", kind="stage", dtype="f16", n=8, h=112, c=64, k=128, convs=2),
        # fourth stage: small pixels, 512 channels
        dict(name="vgg_stage4_b8", kind="stage", dtype="f16", n=8, h=28, c=256, k=512, convs=3),
        # VGG-16's classifier at batch 8: the weights' stream from memory
        dict(name="fc_head_b8", kind="head", dtype="f16", m=8, k=25088, hidden=4096, classes=1000),
        # MobileNetV2's inverted residual at batch 16: expand, depthwise, project + residual
        dict(name="mbv2_block_b16", kind="inverted", dtype="bf16", n=16, h=56, c=24, k=24, expand=6, stride=1),
        # one encoder layer for a single short sequence: many small launches
        dict(name="encoder_b1_s128", kind="encoder", dtype="bf16", batch=1, seq=128, hidden=768, heads=12, ffn=3072),
        # and for a batch of longer ones: large products, attention over 512 tokens
        dict(name="encoder_b8_s512", kind="encoder", dtype="bf16", batch=8, seq=512, hidden=768, heads=12, ffn=3072),
        # a critical ResNet-18 request at batch 1 through the coordinator, until it has completed
        dict(name="request_resnet18", kind="request", dtype="f16", n=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        # no more than the largest listed ones (fp32 runs at a sixteenth of the 16-bit rate)
        if w["bytes"] <= 260e6 and w["flops"] <= (6e9 if case["dtype"] == "f32" else 64e9):
            return case


def _draw(rng):
    kind = rng.choice(["conv", "conv", "conv", "basic", "stage", "stage", "head", "inverted", "inverted", "encoder",
                       "encoder", "request"])
    half = rng.choice(["f16", "bf16"])
    if kind == "conv":
        ks = rng.choice([1, 1, 3, 3, 3, 5, 7])
        stride = rng.choice([1, 1, 2])
        return dict(kind=kind, dtype=rng.choice([half, half, "f32"]), n=_log(rng, 1, 32), h=_log(rng, 7, 160),
                    w=_log(rng, 7, 160), c=rng.choice([8, 24, 32, 40, 64, 72, 96, 128, 192, 256, 320, 512]),
                    k=rng.choice([16, 24, 64, 96, 100, 128, 160, 256, 384, 512]), ks=ks, stride=stride,
                    act=rng.choice(["none", "relu", "relu6"]), bn=rng.random() < 0.5, bias=rng.random() < 0.5,
                    residual=rng.random() < 0.3, shards=rng.choice([1, 1, 2, 3, 4]), block=rng.choice([128, 256, 256, 256]))
    if kind == "basic":
        stride = rng.choice([1, 2])
        c = rng.choice([64, 128, 256] if stride == 2 else [64, 128, 256, 512])
        return dict(kind=kind, dtype=half, n=_log(rng, 1, 16), h=rng.randint(7, 56), c=c, k=c * stride, stride=stride)
    if kind == "stage":
        k = rng.choice([64, 128, 256, 512])
        return dict(kind=kind, dtype=half, n=_log(rng, 1, 16), h=_log(rng, 14, 224), c=8 if k == 64 else k // rng.choice([1, 2]),
                    k=k, convs=rng.choice([2, 3]))
    if kind == "head":
        return dict(kind=kind, dtype=half, m=_log(rng, 1, 64), k=8 * _log(rng, 64, 3136), hidden=8 * _log(rng, 64, 512),
                    classes=rng.randint(10, 1000))
    if kind == "inverted":
        c = rng.choice([16, 24, 32, 64, 96, 160])
        stride = rng.choice([1, 2])
        return dict(kind=kind, dtype=half, n=_log(rng, 1, 32), h=_log(rng, 7, 112), c=c,
                    k=c if stride == 1 else rng.choice([24, 32, 64, 96, 160]), expand=6, stride=stride)
    if kind == "encoder":
        heads = rng.choice([4, 8, 12, 16])
        return dict(kind=kind, dtype=half, batch=_log(rng, 1, 16), seq=_log(rng, 16, 512), hidden=64 * heads, heads=heads,
                    ffn=256 * heads)
    return dict(kind=kind, dtype=half, n=_log(rng, 1, 16))


# ------------------------------------------------------- layers over own buffers
class Layers:
    """The layers of one case: tensors made from the seed on the GPU (or, dry, on no device: shapes
    only), one output buffer and one operator per layer.  Weights and activations have the
    distributions of the framework's network builders."""

    def __init__(self, dtype, seed, dry=False):
        self.dtype, self.dry = TORCH[dtype], dry
        self.dev = "meta" if dry else "cuda"
        self.gen = None if dry else torch.Generator(device="cuda").manual_seed(seed)
        self.steps = []  # (kind, tensors, parameters)
        self.ops = []
        self.outs = []

    def u(self, shape, lo, hi, dtype=None):
        dtype = dtype or self.dtype
        if self.dry:
            return torch.empty(shape, dtype=dtype, device="meta")
        return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=self.gen).to(dtype)

    def buf(self, *shape):
        return torch.empty(shape, dtype=self.dtype, device=self.dev)

    def add(self, kind, y, tensors, params, make):
        self.steps.append((kind, dict(tensors, y=y), params))
        self.outs.append(y)
        if not self.dry:
            self.ops.append(make())
        return y

    def bn(self, c):
        a, b = self.u((2, c), 0.8, 1.2, torch.float32), self.u((2, c), -0.1, 0.1, torch.float32)
        return torch.stack([a[0], b[0], b[1], a[1]])  # gamma, beta, mean, var

    def conv(self, x, k, ks, stride, pad, act, bn=False, bias=False, residual=None, image=False):
        n, h, w, c = x.shape
        fan = (3 if image else c) * ks * ks
        wt = self.u((k, ks, ks, c), -math.sqrt(6 / fan), math.sqrt(6 / fan))
        if image and not self.dry:
            wt[..., 3:] = 0
        b = self.u((k,), -1 / math.sqrt(fan), 1 / math.sqrt(fan), torch.float32) if bias else None
        p = self.bn(k) if bn else None
        y = self.buf(n, (h + 2 * pad - ks) // stride + 1, (w + 2 * pad - ks) // stride + 1, k)
        return self.add("conv", y, dict(x=x, w=wt, bias=b, bn=p, residual=residual), dict(stride=stride, pad=pad, act=act),
                        lambda: ops.conv2d(x, wt, y, stride=stride, pad=pad, bias=b, bn=p, residual=residual, act=act))

    def dwconv(self, x, stride, act):
        n, h, w, c = x.shape
        wt = self.u((3, 3, c), -math.sqrt(6 / 9), math.sqrt(6 / 9))
        p = self.bn(c)
        y = self.buf(n, (h - 1) // stride + 1, (w - 1) // stride + 1, c)
        return self.add("dwconv", y, dict(x=x, w=wt, bn=p), dict(stride=stride, pad=1, act=act),
                        lambda: ops.dwconv(x, wt, y, stride=stride, pad=1, bn=p, act=act))

    def maxpool(self, x, k):
        n, h, w, c = x.shape
        y = self.buf(n, h // k, w // k, c)
        return self.add("maxpool", y, dict(x=x), dict(k=k, stride=k, pad=0), lambda: ops.pool(x, y, k, k, 0, "max"))

    def linear(self, x, nout, act="none", residual=None, bound=None):
        m, k = x.shape
        bound = bound or math.sqrt(6 / k)
        wt = self.u((nout, k), -bound, bound)
        b = self.u((nout,), -1 / math.sqrt(k), 1 / math.sqrt(k), torch.float32)
        y = self.buf(m, nout)
        return self.add("gemm", y, dict(x=x, w=wt, bias=b, residual=residual), dict(act=act),
                        lambda: ops.gemm(x, wt, y, bias=b, residual=residual, act=act))

    def layernorm(self, x, res=None):
        m, n = x.shape
        g, b = self.u((n,), 0.8, 1.2, torch.float32), self.u((n,), -0.1, 0.1, torch.float32)
        y = self.buf(m, n)
        return self.add("layernorm", y, dict(x=x, gamma=g, beta=b), dict(eps=1e-5), lambda: ops.layernorm(x, g, b, y, m, n))

    def attention(self, qkv, B, H, S, D):
        hid = H * D
        at = dict(B=B, H=H, S=S, D=D)
        scores, probs, ctx = self.buf(B * H, S, S), self.buf(B * H, S, S), self.buf(B * S, hid)
        q3, ss = (S * 3 * hid, D), (H * S * S, S * S)
        self.add("scores", scores, dict(x=qkv), at,
                 lambda: ops.bgemm(qkv, qkv[:, hid:], scores, m=S, n=S, k=D, batch=B * H, batch_div=H, ldx=3 * hid,
                                   ldw=3 * hid, ldy=S, sx=q3, sw=q3, sy=ss))
        self.add("softmax", probs, dict(x=scores), dict(scale=1 / math.sqrt(D)),
                 lambda: ops.softmax(scores, probs, B * H * S, S, scale=1 / math.sqrt(D)))
        return self.add("context", ctx, dict(x=probs, w=qkv), at,
                        lambda: ops.bgemm(probs, qkv[:, 2 * hid:], ctx, m=S, n=D, k=S, batch=B * H, batch_div=H, ldx=S,
                                          ldw=3 * hid, ldy=hid, sx=ss, sw=q3, sy=(S * hid, D), b_nmajor=True))


def _layers(case, seed, dry=False):
    L = Layers(case["dtype"], seed, dry)
    kind = case["kind"]
    if kind == "conv":
        x = L.u((case["n"], case["h"], case["w"], case["c"]), -1, 1)
        pad = case["ks"] // 2
        res = None
        if case["residual"]:
            res = L.u((case["n"], (case["h"] + 2 * pad - case["ks"]) // case["stride"] + 1,
                       (case["w"] + 2 * pad - case["ks"]) // case["stride"] + 1, case["k"]), -1, 1)
        L.conv(x, case["k"], case["ks"], case["stride"], pad, case["act"], case["bn"], case["bias"], res)
    elif kind == "basic":
        x = L.u((case["n"], case["h"], case["h"], case["c"]), 0, 2)
        s, k = case["stride"], case["k"]
        ident = x if s == 1 and case["c"] == k else L.conv(x, k, 1, s, 0, "none", bn=True)
        t = L.conv(x, k, 3, s, 1, "relu", bn=True)
        L.conv(t, k, 3, 1, 1, "relu", bn=True, residual=ident)
    elif kind == "stage":
        image = case["c"] == 8
        h = L.u((case["n"], case["h"], case["h"], case["c"]), -1 if image else 0, 1)
        if image and not dry:
            h[..., 3:] = 0
        for _ in range(case["convs"]):
            h = L.conv(h, case["k"], 3, 1, 1, "relu", bias=True, image=image)
            image = False
        L.maxpool(h, 2)
    elif kind == "head":
        h = L.u((case["m"], case["k"]), 0, 1)
        h = L.linear(h, case["hidden"], "relu")
        h = L.linear(h, case["hidden"], "relu")
        L.linear(h, case["classes"])
    elif kind == "inverted":
        x = L.u((case["n"], case["h"], case["h"], case["c"]), -1, 1)
        e = L.conv(x, case["c"] * case["expand"], 1, 1, 0, "relu6", bn=True)
        d = L.dwconv(e, case["stride"], "relu6")
        L.conv(d, case["k"], 1, 1, 0, "none", bn=True, residual=x if case["stride"] == 1 and case["c"] == case["k"] else None)
    elif kind == "encoder":
        B, S, hid, H = case["batch"], case["seq"], case["hidden"], case["heads"]
        x = L.u((B * S, hid), -1, 1)
        bound = 1 / math.sqrt(hid)
        qkv = L.linear(x, 3 * hid, bound=bound)
        ctx = L.attention(qkv, B, H, S, hid // H)
        x1 = L.layernorm(L.linear(ctx, hid, residual=x, bound=bound))
        f = L.linear(x1, case["ffn"], "gelu", bound=bound)
        L.layernorm(L.linear(f, hid, residual=x1, bound=1 / math.sqrt(case["ffn"])))
    else:
        raise ValueError(kind)
    return L


# ------------------------------------------------------------------- requests
class Request:
    """A task of the process's coordinator; the coordinator ends with its last task."""

    coord, users = None, 0

    def __init__(self, net):
        if Request.coord is None:
            Request.coord = Coordinator(policy="elastic")
        Request.users += 1
        self.net = net
        self.task = Request.coord.task(net.ops())

    def run(self):
        co = Request.coord
        co.submit(self.task, True)
        co.drain()
        co.poll(64)

    def __del__(self):
        Request.users -= 1
        if Request.users == 0 and Request.coord is not None:
            Request.coord.shutdown()
            Request.coord = None


def _net(case, seed):
    return models.resnet18(batch=case["n"], dtype=case["dtype"], seed=seed % (1 << 31))


# ------------------------------------------------------------------ the interface
def prepare(case, seed):
    if case["kind"] == "request":
        return Request(_net(case, seed))
    L = _layers(case, seed)
    plan = None
    if case.get("shards", 1) > 1:
        op, s = L.ops[0], min(case["shards"], L.ops[0].T)
        cuts = [j * op.T // s for j in range(s + 1)]
        plan = [(b, e - b, e - b, case["block"]) for b, e in zip(cuts, cuts[1:])]
    elif case.get("block", 256) != 256:
        plan = [(0, L.ops[0].T, L.ops[0].T, case["block"])]
    return dict(layers=L, plan=plan)


def run(state):
    if isinstance(state, Request):
        state.run()
        return {l.name: l.t["y"] for l in state.net.layers}
    L = state["layers"]
    if state["plan"]:
        for shard in state["plan"]:
            L.ops[0].launch(*shard)
    else:
        for op in L.ops:
            op.run()
    return L.outs


_RESNET = [(56, 64, 64, 1, 2), (56, 64, 128, 2, 2), (28, 128, 256, 2, 2), (14, 256, 512, 2, 2)]


def work(case):
    """Inputs and weights read once, outputs written once; multiply-adds as two operations."""
    es = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "request":
        n = case["n"]
        flops = 2 * 112 * 112 * 64 * 147 * n
        weights, acts = 64 * 147, 224 * 224 * 3 + 112 * 112 * 64 + 56 * 56 * 64
        for h, c, k, s, blocks in _RESNET:
            ho = h // s
            acts += ho * ho * k * (2 * blocks + (1 if s == 2 else 0))
            weights += 9 * c * k + 9 * k * k * (2 * blocks - 1) + (c * k if s == 2 else 0)
            flops += 2 * n * ho * ho * (9 * c * k + 9 * k * k * (2 * blocks - 1) + (c * k if s == 2 else 0))
        return dict(bytes=float(es * (weights + 512 * 1000 + n * (acts + 512 + 1000))), flops=float(flops + 2 * n * 512 * 1000))
    L = _layers(case, 0, dry=True)
    flops, made = 0.0, {id(y) for y in L.outs}
    read = {}
    for kind, t, p in L.steps:
        y = t["y"]
        for v in t.values():
            if v is not None and id(v) not in made:
                read[id(v)] = v.numel() * v.element_size()
        if kind == "conv":
            flops += 2.0 * y.numel() * (t["w"].numel() // t["w"].shape[0])
        elif kind == "gemm":
            flops += 2.0 * y.numel() * t["x"].shape[1]
        elif kind in ("scores", "context"):
            flops += 2.0 * p["B"] * p["H"] * p["S"] * p["S"] * p["D"]
        elif kind == "dwconv":
            flops += 18.0 * y.numel()
        else:
            flops += 4.0 * y.numel()
    return dict(bytes=float(sum(read.values()) + es * sum(y.numel() for y in L.outs)), flops=flops)


def tolerance(case):
    """About four times what the layers differ by from their float64 values: one layer 2.1e-4 (f16)
    and 1.7e-3 (bf16), the last of a block's or a network's layers up to 7e-4 and 3.3e-3; fp32 sums
    4e-7 at K = 576, more at the longest K drawn."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    ulp = 2.0 ** -10 if case["dtype"] == "f16" else 2.0 ** -7  # two roundings of one value apart
    if case["kind"] == "conv":
        return {"rel": 0.9 * ulp, "max": 4 * ulp}
    return {"rel": (2.5 if case["dtype"] == "f16" else 1.7) * ulp, "max": 16 * ulp}


# ------------------------------------------------------------------ float64 values
def _act(v, act):
    if act == "relu":
        return v.clamp_(min=0)
    if act == "relu6":
        return v.clamp_(0, 6)
    if act == "gelu":
        return 0.5 * v * (1 + torch.special.erf(v / math.sqrt(2.0)))
    return v


def _epilogue(v, t, p, get):
    if t.get("bias") is not None:
        v = v + t["bias"].double()
    if t.get("bn") is not None:
        g, b, mu, var = t["bn"].double()
        v = (v - mu) * (g / torch.sqrt(var + p.get("eps", 1e-5))) + b
    if t.get("residual") is not None:
        v = v + get(t["residual"]).reshape(v.shape)
    return _act(v, p["act"])


def _value(kind, t, p, get):
    x, shape = get(t["x"]), t["y"].shape
    if kind in ("conv", "dwconv"):
        w, s, pad = t["w"].double(), p["stride"], p["pad"]
        kh, kw = (w.shape[1], w.shape[2]) if kind == "conv" else (3, 3)
        n, ho, wo, k = shape
        xp = F.pad(x, (0, 0, pad, pad, pad, pad))
        v = torch.zeros((n, ho, wo, k), dtype=torch.float64, device=x.device)
        for r in range(kh):
            for c in range(kw):
                tap = xp[:, r:r + s * (ho - 1) + 1:s, c:c + s * (wo - 1) + 1:s, :]
                v += tap @ w[:, r, c, :].t().contiguous() if kind == "conv" else tap * w[r, c]
        return _epilogue(v, t, p, get)
    if kind == "gemm":
        return _epilogue(x.reshape(shape[0], -1) @ t["w"].double().t(), t, p, get)
    if kind in ("maxpool", "avgpool"):
        f = F.max_pool2d if kind == "maxpool" else F.avg_pool2d
        return f(x.permute(0, 3, 1, 2), p["k"], p["stride"], p["pad"]).permute(0, 2, 3, 1)
    if kind == "layernorm":
        return F.layer_norm(x, (x.shape[1],), t["gamma"].double(), t["beta"].double(), p["eps"])
    if kind == "softmax":
        return torch.softmax(x * p["scale"], -1)
    B, H, S, D = p["B"], p["H"], p["S"], p["D"]
    q, k, v = (get(t["w"]) if kind == "context" else x).reshape(B, S, 3, H, D).permute(2, 0, 3, 1, 4).reshape(3, B * H, S, D)
    if kind == "scores":
        return torch.bmm(q.contiguous(), k.transpose(1, 2).contiguous())
    return torch.bmm(x, v.contiguous()).reshape(B, H, S, D).permute(0, 2, 1, 3).reshape(B * S, H * D)


def _float64(steps):
    """float64 values of every layer's output, each from the float64 values of the layers before it."""
    known = {}

    def get(t):
        v = known.get(t.data_ptr())  # a layer's output, under any view of its buffer
        return v.reshape(t.shape) if v is not None else t.double()

    outs = []
    for kind, t, p in steps:
        v = _value(kind, t, p, get).reshape(t["y"].shape)
        known[t["y"].data_ptr()] = v
        outs.append(v)
    return outs


def exact(case, seed):
    if case["kind"] == "request":
        net = _net(case, seed)
        return dict(zip((l.name for l in net.layers), _float64([(l.kind, l.t, l.params) for l in net.layers])))
    return _float64(_layers(case, seed).steps)
