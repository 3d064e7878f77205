"""Performance cases: inference through pruned layers, blocks and whole stacks, by the public entry points.

A case is a dict of plain values.  `kind` names the call a program makes:

  conv       one block-punched convolution        npas.conv2d_sparse   (k = 1, 3, 5; stride 1 or 2; 16-bit or fp32)
  pattern    one pattern + kernel-removal 3x3      npas.conv2d_sparse
  fc         one block-based sparse FC layer       npas.fc_sparse
  depthwise  one depthwise 3x3 layer               npas.depthwise3x3
  pair       1x1 -> act -> 1x1                     npas.Stack.run, fusion allowed
  block      1x1 -> depthwise 3x3 -> 1x1 (+ x)     npas.Stack.run, fusion allowed
  residual   bottleneck residual network           npas.Stack.run, all fusions allowed (a whole call; returns the logits)

Activations are ~N(0, 1), weights N(0, 2 rate / fan-in), masks have the structure of the scheme, all drawn on the GPU from
the seed.  Packed handles, stacks, outputs and workspaces are made once in `prepare`, as a serving program makes them.
"""
import math

import numpy as np
import torch

import paper_2012_00596_amd as npas

DTYPES = {"f32": (npas.F32, torch.float32), "bf16": (npas.BF16, torch.bfloat16), "f16": (npas.F16, torch.float16)}
ACTS = {"none": npas.ACT_NONE, "relu": npas.ACT_RELU, "relu6": npas.ACT_RELU6, "hswish": npas.ACT_HARDSWISH}


def listed():
    return [
        # The smallest call: one fp32 layer on one small image, where launch and latency count.
        dict(name="conv3x3_f32_b1", kind="conv", dtype="f32", N=1, H=32, W=32, C=16, F=32, k=3, stride=1, act="none",
             bias=False, res=False, Bf=4, Bc=4, rate=2),
        # Pointwise layers of the residual network in its widest form: expansion with the shortcut added.
        dict(name="conv1x1_expand_b128", kind="conv", dtype="bf16", N=128, H=14, W=14, C=256, F=1024, k=1, stride=1,
             act="relu", bias=True, res=True, Bf=8, Bc=4, rate=2),
        # A mobile network's projection run as its own layer: few channels that are no multiple of 64, odd maps, fp16.
        dict(name="conv1x1_ragged_f16", kind="conv", dtype="f16", N=64, H=57, W=57, C=144, F=40, k=1, stride=1,
             act="hswish", bias=True, res=False, Bf=8, Bc=8, rate=4),
        # The 3x3 layer in the middle of a bottleneck block, a full serving batch.
        dict(name="conv3x3_b128", kind="conv", dtype="bf16", N=128, H=14, W=14, C=256, F=256, k=3, stride=1, act="relu",
             bias=False, res=False, Bf=8, Bc=4, rate=3),
        # The downsampling 3x3 layer at the head of a stage, a middling batch.
        dict(name="conv3x3_s2_b32", kind="conv", dtype="bf16", N=32, H=56, W=56, C=128, F=128, k=3, stride=2, act="relu",
             bias=True, res=False, Bf=8, Bc=4, rate=3),
        # Pattern-pruned 3x3 layer (4 of 9 taps, 30 % of the kernels removed).
        dict(name="pattern3x3_b32", kind="pattern", dtype="bf16", N=32, H=28, W=28, C=128, F=128, act="none", bias=False,
             dead=0.3),
        # Block-based sparse classifier.
        dict(name="fc_b256", kind="fc", dtype="bf16", N=256, C=1280, F=1000, act="none", bias=True, Bf=16, Bc=32, rate=5),
        # Depthwise layer of a mobile network on its own, odd maps.
        dict(name="depthwise_b32", kind="depthwise", dtype="bf16", N=32, H=57, W=57, C=144, stride=1, act="relu6", bias=True),
        # Expansion and projection without the depthwise layer between them, as one stack call.
        dict(name="pair_b64", kind="pair", dtype="bf16", N=64, H=56, W=56, C=24, mid=144, act="relu6", Bf=8, Bc=8, rate=4),
        # The inverted-residual block of a mobile network with folded batch norms.
        dict(name="block_b64", kind="block", dtype="bf16", N=64, H=56, W=56, C=24, mid=144, stride=1, act="relu6", bias=True,
             Bf=8, Bc=8, rate=4),
        # The whole 50-layer network on one image (interactive use) and on a full batch (throughput).
        dict(name="residual50_b1", kind="residual", dtype="bf16", N=1, HW=224, width=64, stages=50, classes=1000),
        dict(name="residual50_b128", kind="residual", dtype="bf16", N=128, HW=224, width=64, stages=50, classes=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv1", "conv1", "conv3", "conv3", "conv_f32", "pattern", "fc", "depthwise", "pair", "block", "residual"])
    dt = rng.choice(["bf16", "bf16", "f16"])
    if kind == "conv_f32":
        return dict(kind="conv", dtype="f32", N=rng.randint(1, 4), H=rng.randint(8, 40), W=rng.randint(8, 40),
                    C=rng.randint(3, 48), F=rng.randint(8, 64), k=rng.choice([1, 3, 5]), stride=rng.choice([1, 1, 2]),
                    act=rng.choice(["none", "relu"]), bias=rng.random() < 0.5, res=False, Bf=4, Bc=4,
                    rate=rng.choice([2, 3, 5]))
    if kind in ("conv1", "conv3"):
        HW = rng.choice([7, 14, 28, 56, rng.randint(7, 60)])
        wide = rng.random() < 0.6   # residual-network widths, or a mobile network's (multiples of 8, now and then of 4)
        if wide:
            C, F = 64 * _log_int(rng, 1, 16 if kind == "conv1" else 8), 64 * _log_int(rng, 1, 16 if kind == "conv1" else 8)
        else:
            C, F = 8 * _log_int(rng, 2, 40), 4 * _log_int(rng, 4, 80)
        k = 1 if kind == "conv1" else 3
        stride = rng.choice([1, 1, 1, 2])
        N = _log_int(rng, 1, 128)
        while N > 1 and N * HW * HW * max(C, F) > 128 * 56 * 56 * 256 // 2:   # no more than the widest layers of the network
            N //= 2
        return dict(kind="conv", dtype=dt, N=N, H=HW, W=max(3, HW - rng.choice([0, 0, 1])), C=C, F=F, k=k, stride=stride,
                    act=rng.choice(["none", "relu", "relu6", "hswish"]), bias=rng.random() < 0.5,
                    res=stride == 1 and rng.random() < 0.4, Bf=8, Bc=rng.choice([4, 8]), rate=rng.choice([2, 3, 5]))
    if kind == "pattern":
        return dict(kind="pattern", dtype=dt, N=_log_int(rng, 1, 64), H=rng.randint(7, 56), W=rng.randint(7, 56),
                    C=rng.choice([64, 128, 192, 256]), F=rng.choice([64, 128, 192, 256]), act=rng.choice(["none", "relu"]),
                    bias=rng.random() < 0.5, dead=rng.choice([0.0, 0.3, 0.5]))
    if kind == "fc":
        return dict(kind="fc", dtype=dt, N=_log_int(rng, 1, 1024), C=64 * rng.randint(4, 40), F=4 * rng.randint(16, 500),
                    act="none", bias=rng.random() < 0.5, Bf=16, Bc=32, rate=rng.choice([2, 3, 5]))
    if kind == "depthwise":
        return dict(kind="depthwise", dtype=dt, N=_log_int(rng, 1, 64), H=rng.randint(7, 60), W=rng.randint(7, 60),
                    C=8 * _log_int(rng, 2, 60), stride=rng.choice([1, 2]), act=rng.choice(["relu6", "hswish"]),
                    bias=rng.random() < 0.5)
    if kind in ("pair", "block"):
        C = 8 * rng.randint(2, 4)
        c = dict(kind=kind, dtype=dt, N=_log_int(rng, 1, 96), H=rng.randint(7, 60), W=rng.randint(7, 60), C=C,
                 mid=C * rng.choice([3, 4, 6]), act=rng.choice(["relu6", "relu6", "hswish"]), Bf=8, Bc=8,
                 rate=rng.choice([2, 4]))
        if kind == "block":
            c.update(stride=rng.choice([1, 1, 2]), bias=rng.random() < 0.5)
        return c
    return dict(kind="residual", dtype=dt, N=_log_int(rng, 1, 64), HW=32 * rng.randint(2, 7), width=64, stages=rng.choice([14, 26]),
                classes=100 * rng.randint(1, 10))


# ---- inputs ------------------------------------------------------------------

def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _keep_smallest(keys, counts):
    """0/1 tensor: per row the counts[row] smallest keys."""
    rank = keys.argsort(dim=1).argsort(dim=1)
    return rank < counts[:, None]


def _punched_mask(g, F, C, k, Bf, Bc, rate):
    """Block-punched mask [F][C][k][k]: per Bf x Bc block 1/rate of the positions kept, the same in all its filters."""
    G, NB, T = -(-F // Bf), -(-C // Bc), k * k
    keys = torch.rand((G * NB, Bc * T), generator=g, device="cuda")
    sizes = torch.full((NB,), Bc * T, device="cuda")
    sizes[-1] = (C - (NB - 1) * Bc) * T
    exists = torch.arange(Bc * T, device="cuda")[None, :] < sizes.repeat(G)[:, None]
    cum = torch.nn.functional.pad(sizes.repeat(G).cumsum(0), (1, 0)) // rate
    keep = _keep_smallest(torch.where(exists, keys, 2.0), cum[1:] - cum[:-1]) & exists
    return keep.reshape(G, NB * Bc, k, k)[:, :C].repeat_interleave(Bf, dim=0)[:F].contiguous()


def _pattern_mask(g, F, C, dead):
    """Every 3x3 kernel keeps the centre and three more taps (one of 8 patterns); a share `dead` of the kernels is removed."""
    combos = [(a, b, c) for a in range(8) for b in range(a + 1, 8) for c in range(b + 1, 8)]
    pick = torch.randperm(len(combos), generator=g, device="cuda")[:8].sort().values.tolist()
    lib = np.zeros((8, 9), dtype=np.uint8)
    for i, p in enumerate(pick):
        lib[i, 4] = 1
        lib[i, [(0, 1, 2, 3, 5, 6, 7, 8)[t] for t in combos[p]]] = 1
    ids = torch.randint(0, 8, (F * C,), generator=g, device="cuda")
    mask = torch.from_numpy(lib).cuda().bool()[ids]
    order = torch.rand(F * C, generator=g, device="cuda").argsort()
    mask[order[:int(dead * F * C + 0.5)]] = False
    return mask.reshape(F, C, 3, 3), lib


class _Layer:
    """One layer of a case: its weights (storage type), mask and wiring."""

    def __init__(self, op, C=0, F=0, k=1, stride=1, pad=0, act="none", src=0, res=-1, w=None, mask=None, lib=None, block=(1, 1),
                 bias=None):
        self.op, self.C, self.F, self.k, self.stride, self.pad, self.act = op, C, F, k, stride, pad, act
        self.src, self.res, self.w, self.mask, self.lib, self.block, self.bias = src, res, w, mask, lib, block, bias

    def pack(self, dtype):
        code, td = DTYPES[dtype]
        w = self.w.cpu()
        w = w.numpy() if td == torch.float32 else w.view(torch.int16).numpy().view(np.uint16)
        if self.op == "depthwise":
            return npas.pack_depthwise3x3(w, code)
        m = self.mask.to(torch.uint8).cpu().numpy()
        if self.op == "pattern":
            return npas.pack_pattern(w, m, self.lib, code)
        if self.op == "fc":
            return npas.pack_fc_block(w.reshape(self.F, self.C), m.reshape(self.F, self.C), *self.block, code)
        return npas.pack_block_punched(w, m, *self.block, code)


def _punched(g, td, C, F, k, stride, act, src, block, rate, res=-1, bias=False, scale=1.0, op="conv"):
    w = (_randn(g, F, C, k, k) * (scale * math.sqrt(2.0 * rate / (C * k * k)))).to(td)
    return _Layer(op, C, F, k, stride, k // 2, act, src, res, w, _punched_mask(g, F, C, k, *block, rate), block=block,
                  bias=_randn(g, F) * 0.5 if bias else None)


def _depthwise(g, td, C, stride, act, src, bias):
    return _Layer("depthwise", C, C, 3, stride, 1, act, src, w=(_randn(g, C, 3, 3) / 3.0).to(td),
                  bias=_randn(g, C) * 0.5 if bias else None)


_STAGES = {50: (3, 4, 6, 3), 26: (2, 2, 2, 2), 14: (1, 1, 1, 1)}


def _residual_layers(g, td, case):
    width, layers = case["width"], []

    def conv(C, F, k, stride, act, src, res=-1, scale=1.0):
        rate = (2, 3, 5)[int(torch.randint(0, 3, (1,), generator=g, device="cuda"))]
        layers.append(_punched(g, td, C, F, k, stride, act, src, (8, 4), rate, res, scale=scale))
        return len(layers)

    conv(3, width, 7, 2, "relu", 0)
    layers.append(_Layer("maxpool", width, width, 3, 2, 1, src=1))
    t, cin = 2, width
    for s, n in enumerate(_STAGES[case["stages"]]):
        mid = width << s
        for b in range(n):
            stride = 2 if b == 0 and s > 0 else 1
            a = conv(cin, mid, 1, 1, "relu", t)
            a = conv(mid, mid, 3, stride, "relu", a)
            sc = conv(cin, 4 * mid, 1, stride, "none", t) if b == 0 else t
            t, cin = conv(mid, 4 * mid, 1, 1, "relu", a, res=sc, scale=0.25), 4 * mid
    layers.append(_Layer("avgpool", cin, cin, src=t))
    layers.append(_punched(g, td, cin, case["classes"], 1, 1, "none", len(layers), (16, 32), 3, op="fc", scale=0.7))
    return layers


def _make(case, seed):
    """(x, residual or None, layers) of a case, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    td, kind = DTYPES[case["dtype"]][1], case["kind"]
    res = None
    if kind == "residual":
        x = _randn(g, case["N"], case["HW"], case["HW"], 3).to(td)
        return x, None, _residual_layers(g, td, case)
    if kind == "fc":
        x = _randn(g, case["N"], case["C"]).to(td)
    else:
        x = _randn(g, case["N"], case["H"], case["W"], case["C"]).to(td)
    block = (case.get("Bf"), case.get("Bc"))
    if kind in ("conv", "fc"):
        layers = [_punched(g, td, case["C"], case["F"], case.get("k", 1), case.get("stride", 1), case["act"], 0, block, case["rate"],
                           bias=case["bias"], op=kind)]
        if case.get("res"):
            res = _randn(g, *_out_shape(layers[0], x.shape)).to(td)
    elif kind == "pattern":
        C, F = case["C"], case["F"]
        mask, lib = _pattern_mask(g, F, C, case["dead"])
        w = (_randn(g, F, C, 3, 3) * math.sqrt(2.0 / (4 * C))).to(td)
        layers = [_Layer("pattern", C, F, 3, 1, 1, case["act"], 0, w=w, mask=mask, lib=lib,
                         bias=_randn(g, F) * 0.5 if case["bias"] else None)]
    elif kind == "depthwise":
        layers = [_depthwise(g, td, case["C"], case["stride"], case["act"], 0, case["bias"])]
    else:
        C, mid, act, rate, bias = case["C"], case["mid"], case["act"], case["rate"], case.get("bias", False)
        layers = [_punched(g, td, C, mid, 1, 1, act, 0, block, rate, bias=bias)]
        if kind == "block":
            layers.append(_depthwise(g, td, mid, case["stride"], act, 1, bias))
        layers.append(_punched(g, td, mid, C, 1, 1, "none", len(layers), block, rate, bias=bias,
                               res=0 if kind == "block" and case["stride"] == 1 else -1))
    return x, res, layers


def _out_shape(L, s):
    if L.op == "fc":
        return (s[0], L.F)
    if L.op == "avgpool":
        return (s[0], s[3])
    return (s[0], (s[1] + 2 * L.pad - L.k) // L.stride + 1, (s[2] + 2 * L.pad - L.k) // L.stride + 1, L.F)


def _shapes(x_shape, layers):
    shapes = [tuple(x_shape)]
    for L in layers:
        shapes.append(_out_shape(L, shapes[L.src]))
    return shapes


# ---- the measured call -------------------------------------------------------

def prepare(case, seed):
    x, res, layers = _make(case, seed)
    td = DTYPES[case["dtype"]][1]
    state = {"kind": case["kind"], "x": x, "res": res, "layer": layers[0], "act": ACTS[layers[0].act], "bias": layers[0].bias,
             "y": torch.empty(_shapes(x.shape, layers)[-1], dtype=td, device="cuda")}
    packed = [L.pack(case["dtype"]) if L.w is not None else None for L in layers]
    state["packed"] = packed[0]
    if case["kind"] in ("pair", "block", "residual"):
        kinds = {"conv": npas.LAYER_CONV, "fc": npas.LAYER_FC, "maxpool": npas.LAYER_MAXPOOL3X3S2,
                 "avgpool": npas.LAYER_GLOBAL_AVGPOOL, "depthwise": npas.LAYER_DEPTHWISE3X3}
        stack = npas.Stack([dict(kind=kinds[L.op], packed=p, stride=L.stride, pad=L.pad, act=ACTS[L.act], src=L.src, res=L.res,
                                 bias=L.bias) for L, p in zip(layers, packed)], x.shape[1], x.shape[2],
                           npas.STACK_FUSE_POINTWISE | npas.STACK_FUSE_INVERTED_RESIDUAL | npas.STACK_FUSE_CONV_MAXPOOL)
        state["stack"], state["biases"], state["bytes"] = stack, [L.bias for L in layers], stack.workspace_bytes(x.shape[0])
        state["workspace"] = torch.empty(max(state["bytes"], 256), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    s, x, y, kind = torch.cuda.current_stream().cuda_stream, state["x"], state["y"], state["kind"]
    if kind in ("conv", "pattern"):
        L = state["layer"]
        npas.conv2d_sparse(state["packed"], x, y, x.shape[0], x.shape[1], x.shape[2], L.stride, L.pad, state["bias"], state["res"],
                           state["act"], s)
    elif kind == "fc":
        npas.fc_sparse(state["packed"], x, y, x.shape[0], state["bias"], state["act"], s)
    elif kind == "depthwise":
        npas.depthwise3x3(state["packed"], x, y, x.shape[0], x.shape[1], x.shape[2], state["layer"].stride, state["bias"], None,
                          state["act"], s)
    else:
        state["stack"].run(x, y, x.shape[0], state["workspace"], state["bytes"], s)
    return y


# ---- what a pass cannot do without -------------------------------------------

def _plan(case):
    """(rate or dead share, geometry) of every layer without making tensors: [(op, C, F, k, stride, src, kept share)], x shape."""
    kind = case["kind"]
    if kind == "residual":
        ops = [("conv", 3, case["width"], 7, 2, 0), ("maxpool", case["width"], case["width"], 3, 2, 1)]
        t, cin = 2, case["width"]
        for s, n in enumerate(_STAGES[case["stages"]]):
            mid = case["width"] << s
            for b in range(n):
                stride, block_in = (2 if b == 0 and s > 0 else 1), t
                ops.append(("conv", cin, mid, 1, 1, block_in))
                ops.append(("conv", mid, mid, 3, stride, len(ops)))
                a = len(ops)
                if b == 0:
                    ops.append(("conv", cin, 4 * mid, 1, stride, block_in))
                ops.append(("conv", mid, 4 * mid, 1, 1, a))
                t, cin = len(ops), 4 * mid
        ops.append(("avgpool", cin, cin, 1, 1, t))
        ops.append(("fc", cin, case["classes"], 1, 1, len(ops)))
        # rates are drawn uniformly from 2, 3, 5: the mean kept share
        return [o + ((1 / 2 + 1 / 3 + 1 / 5) / 3 if o[0] == "conv" else 1 / 3,) for o in ops], (case["N"], case["HW"], case["HW"], 3)
    x = (case["N"], case["C"]) if kind == "fc" else (case["N"], case["H"], case["W"], case["C"])
    if kind in ("conv", "fc"):
        return [(kind, case["C"], case["F"], case.get("k", 1), case.get("stride", 1), 0, 1 / case["rate"])], x
    if kind == "pattern":
        return [("conv", case["C"], case["F"], 3, 1, 0, (1 - case["dead"]) * 4 / 9)], x
    if kind == "depthwise":
        return [("depthwise", case["C"], case["C"], 3, case["stride"], 0, 1.0)], x
    ops = [("conv", case["C"], case["mid"], 1, 1, 0, 1 / case["rate"])]
    if kind == "block":
        ops.append(("depthwise", case["mid"], case["mid"], 3, case["stride"], 1, 1.0))
    return ops + [("conv", case["mid"], case["C"], 1, 1, len(ops), 1 / case["rate"])], x


def work(case):
    """Input, added tensor and output once, the kept weights once; the kept multiply-adds (two operations each)."""
    ops, x = _plan(case)
    size = 4 if case["dtype"] == "f32" else 2
    shapes, elems, flops = [x], math.prod(x), 0
    for op, C, F, k, stride, src, kept in ops:
        s = _out_shape(_Layer(op, C, F, k, stride, k // 2), shapes[src])
        shapes.append(s)
        if op in ("conv", "fc"):
            elems += C * F * k * k * kept
            flops += 2 * math.prod(s) * C * k * k * kept
        elif op == "depthwise":
            elems += 9 * C
            flops += 2 * math.prod(s) * 9
    elems += math.prod(shapes[-1]) * (2 if case.get("res") else 1)
    return {"bytes": int(elems * size), "flops": int(flops)}


def tolerance(case):
    """About four times the distance measured from 64-bit results (fp16: an eighth of bf16's, three more significand bits)."""
    if case["dtype"] == "f32":          # sums are correctly rounded: half a step of the result, 2.6e-8 in the norm
        return {"rel": 1.1e-7, "max": 2.5e-7}
    unit = 1.0 if case["dtype"] == "bf16" else 0.125
    if case["kind"] == "residual":      # a rounding to storage after every layer: 2.7e-3, 9.9e-3
        return {"rel": 1.1e-2 * unit, "max": 4e-2 * unit}
    if case["kind"] in ("pair", "block"):   # one or two rounded tensors between the layers: 2.8e-3, 2.4e-2
        return {"rel": 1.1e-2 * unit, "max": 9e-2 * unit}
    return {"rel": 7e-3 * unit, "max": 1.6e-2 * unit}   # one rounding of the result: 1.7e-3, 3.9e-3


# ---- 64-bit results ----------------------------------------------------------

def _conv64(L, x):
    """Masked convolution in float64 as one matrix product per tap; x [N][H][W][C]."""
    N, H, W, C = x.shape
    w = L.w.double() * L.mask
    xp = torch.nn.functional.pad(x, (0, 0, L.pad, L.pad, L.pad, L.pad))
    _, Ho, Wo, _ = _out_shape(L, x.shape)
    y = torch.zeros((N * Ho * Wo, L.F), dtype=torch.float64, device=x.device)
    for i in range(L.k):
        for j in range(L.k):
            tap = xp[:, i:i + (Ho - 1) * L.stride + 1:L.stride, j:j + (Wo - 1) * L.stride + 1:L.stride]
            y += tap.reshape(-1, C) @ w[:, :, i, j].t()
    return y.reshape(N, Ho, Wo, L.F)


def _depthwise64(L, x):
    N, H, W, C = x.shape
    _, Ho, Wo, _ = _out_shape(L, x.shape)
    w, xp = L.w.double(), torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return sum(xp[:, i:i + (Ho - 1) * L.stride + 1:L.stride, j:j + (Wo - 1) * L.stride + 1:L.stride] * w[:, i, j]
               for i in range(3) for j in range(3))


def _act64(v, act):
    if act == "relu":
        return v.clamp(min=0)
    if act == "relu6":
        return v.clamp(0, 6)
    return v * (v + 3).clamp(0, 6) / 6 if act == "hswish" else v


def exact(case, seed):
    x, res, layers = _make(case, seed)
    last = {L.src: i for i, L in enumerate(layers)}
    last.update({L.res: max(i, last.get(L.res, 0)) for i, L in enumerate(layers) if L.res >= 0})
    t = {0: x.double()}
    for i, L in enumerate(layers):
        v = t[L.src]
        if L.op in ("conv", "pattern"):
            v = _conv64(L, v)
        elif L.op == "fc":
            v = v @ (L.w.double() * L.mask).reshape(L.F, L.C).t()
        elif L.op == "depthwise":
            v = _depthwise64(L, v)
        elif L.op == "maxpool":
            v = torch.nn.functional.pad(v, (0, 0, 1, 1, 1, 1), value=-math.inf)
            _, Ho, Wo, _ = _out_shape(L, t[L.src].shape)
            v = torch.stack([v[:, a:a + 2 * Ho - 1:2, b:b + 2 * Wo - 1:2] for a in range(3) for b in range(3)]).amax(0)
        else:
            v = v.mean((1, 2))
        if L.bias is not None:
            v = v + L.bias.double()
        if L.res >= 0:
            v = v + t[L.res]
        elif res is not None:
            v = v + res.double()
        t[i + 1] = _act64(v, L.act)
        for k in [k for k in t if k <= i and last.get(k, -1) <= i]:
            del t[k]
    return t[len(layers)]
