"""The convolutions this library is timed on, through its public entry points.

A case is one of

  conv    ``Plan.conv2d`` on one layer with its weights transformed once (a
          network's layer in a serving loop), on a tile and a precision,
  weights ``Plan.set_weights`` and ``Plan.conv2d``: a layer whose weights have
          just changed (a network in training, a layer used once),
  noalloc ``conv2d_noalloc``: a call without a plan, which transforms the
          weights itself,
  stack   a chain of ``Plan.conv2d`` calls, each on the output of the one
          before it (a whole super-resolution network).

Inputs are fp32, as the library takes them: images or activations (uniform in
[0, 1] or normal) and weights with fan-in scaling.
"""
import math

import torch

from paper_2102_13272_amd import nwg

AUTO, F23 = nwg.NWG_TILE_AUTO, nwg.NWG_TILE_F2X2_3X3


def _case(name, kind, B, M, N, H, W, r, pad, tile=AUTO, depthwise=False, split=False,
          x_dist="normal"):
    c = dict(kind=kind, B=B, M=M, N=N, H=H, W=W, r=r, pad=pad, tile=tile, depthwise=depthwise,
             split=split, x_dist=x_dist)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest kernel the method is for, on a tiny map: launches and host time
        _case("r4 4-4 16x16 valid", "conv", 1, 4, 4, 16, 16, 4, 0, tile=F23),
        # one 7x7 layer of a small network at batch 1
        _case("r7 32-32 64x64", "conv", 1, 32, 32, 64, 64, 7, 3),
        # a 9x9 layer with many channels (one nesting level of F(3,3) fewer)
        _case("r9 128-128 56x56 b16", "conv", 16, 128, 128, 56, 56, 9, 4),
        # odd sizes everywhere, on the tile a plan takes by default
        _case("r11 48-80 45x61 b3", "conv", 3, 48, 80, 45, 61, 11, 5, tile=F23),
        # a 13x13 layer of a large-kernel backbone
        _case("r13 64-64 56x56 b8", "conv", 8, 64, 64, 56, 56, 13, 6),
        # the 31x31 layer of a large-kernel backbone, the largest kernel served
        _case("r31 128-128 56x56 b16", "conv", 16, 128, 128, 56, 56, 31, 15),
        # the same layer in the 16-bit matrix arithmetic a plan can be set to
        _case("r31 bf16 split b16", "conv", 16, 128, 128, 56, 56, 31, 15, tile=F23, split=True),
        # depthwise layers: 7x7 as in mobile networks, 31x31 as in large-kernel backbones
        _case("dw7 54 83x83 b8", "conv", 8, 54, 54, 83, 83, 7, 3, depthwise=True),
        _case("dw31 128 56x56 b16", "conv", 16, 128, 128, 56, 56, 31, 15, depthwise=True),
        # new weights before the call
        _case("r17 new weights b8", "weights", 8, 64, 64, 56, 56, 17, 8),
        # a small layer in a loop that may not allocate
        _case("noalloc r5 16-16 64x64", "noalloc", 1, 16, 16, 64, 64, 5, 2),
        # a super-resolution network: 8 layers on 4 images, most with few channels
        dict(name="sr stack 256x256 b4", kind="stack", B=4, H=256, W=256, x_dist="uniform_01"),
    ]


# the network of the stack case: (input channels, output channels, kernel size)
STACK = [(1, 32, 5), (32, 5, 1), (5, 5, 3), (5, 5, 3), (5, 5, 3), (5, 5, 3), (5, 32, 1),
         (32, 1, 9)]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _geometry(c):
    if c["depthwise"]:
        return nwg.plan_geometry_depthwise(c["B"], c["M"], c["H"], c["W"], c["r"], c["pad"],
                                           c["tile"])
    return nwg.plan_geometry(c["B"], c["M"], c["N"], c["H"], c["W"], c["r"], c["pad"], c["tile"])


def draw(rng):
    """A case of the listed kinds: kernels of 2 to 31 taps, 1 to 16 images, 1 to 256 channels, maps
    of 8 to 256 values a side, no more memory or matrix work than half the 31x31 layer's."""
    while True:
        u = rng.random()
        if u < 0.06:
            c = dict(kind="stack", B=rng.randint(1, 4), H=_log_int(rng, 32, 256),
                     W=_log_int(rng, 32, 256), x_dist="uniform_01")
            return c
        kind = "noalloc" if u < 0.14 else "weights" if u < 0.22 else "conv"
        depthwise = kind == "conv" and u > 0.82
        split = kind == "conv" and 0.22 <= u < 0.29
        r = _log_int(rng, 2, 31)
        pad = rng.choice([(r - 1) // 2, (r - 1) // 2, (r - 1) // 2, 0])
        B = _log_int(rng, 1, 16)
        M, N = _log_int(rng, 1, 256), _log_int(rng, 1, 256)
        if rng.random() < 0.5:              # whole blocks of channels, as most networks have
            M, N = 16 * max(1, M // 16), 16 * max(1, N // 16)
        if split:
            M, N = 32 * max(1, M // 32), 64 * max(1, N // 64)
        if depthwise:
            N = M
        H = _log_int(rng, 8, 256)
        W = H if rng.random() < 0.4 else _log_int(rng, 8, 256)
        if min(H, W) + 2 * pad < r + 4:
            continue
        tile = F23 if split or rng.random() < 0.35 else AUTO
        c = _case(None, kind, B, M, N, H, W, r, pad, tile, depthwise, split,
                  rng.choice(["normal", "uniform_01"]))
        try:
            g = _geometry(c)
        except nwg.NwgError:
            continue
        if g["workspace_bytes"] > 3.2e9 or g["contract_flop"] > 5e10 or B * M * H * W > 3e7 or \
                B * N * H * W > 3e7 or (depthwise and g["direct_flop"] > 1.2e10):
            continue
        if split and g["T"] < 64:
            continue
        if kind == "noalloc" and g["workspace_bytes"] > nwg.NWG_NOALLOC_SCRATCH_BYTES - 4096:
            continue
        return c


def _layers(c):
    if c["kind"] == "stack":
        return [_case(None, "conv", c["B"], m, n, c["H"], c["W"], r, (r - 1) // 2,
                      x_dist=c["x_dist"]) for m, n, r in STACK]
    return [c]


def _inputs(c, seed):
    """x and the weights of each layer, on the GPU, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    layers = _layers(c)
    shape = (c["B"], layers[0]["M"], c["H"], c["W"])
    make = torch.randn if c["x_dist"] == "normal" else torch.rand
    x = make(shape, generator=gen, device="cuda")
    ws = []
    for s in layers:
        m = 1 if s["depthwise"] else s["M"]
        w = torch.randn((s["N"], m, s["r"], s["r"]), generator=gen, device="cuda")
        ws.append(w * (m * s["r"] * s["r"]) ** -0.5)
    return x, ws


def _out_shape(s):
    return (s["B"], s["N"], s["H"] + 2 * s["pad"] - s["r"] + 1, s["W"] + 2 * s["pad"] - s["r"] + 1)


def prepare(case, seed):
    x, ws = _inputs(case, seed)
    layers = _layers(case)
    ys = [torch.empty(_out_shape(s), device="cuda") for s in layers]
    plans = []
    if case["kind"] != "noalloc":
        for s, w in zip(layers, ws):
            p = nwg.Plan(s["B"], s["M"], s["N"], s["H"], s["W"], s["r"], s["pad"], tile=s["tile"],
                         depthwise=s["depthwise"])
            if s["split"]:
                p.set_precision(nwg.NWG_PRECISION_BF16_SPLIT)
            if case["kind"] != "weights":
                p.set_weights(w)
            plans.append(p)
    return dict(case=case, x=x, ws=ws, ys=ys, plans=plans)


def run(state):
    kind, ws, ys, plans = state["case"]["kind"], state["ws"], state["ys"], state["plans"]
    if kind == "noalloc":
        c = state["case"]
        nwg.conv2d_noalloc(state["x"], ws[0], ys[0], c["pad"], c["tile"])
        return ys[0]
    if kind == "weights":
        plans[0].set_weights(ws[0])
    x = state["x"]
    for p, w, y in zip(plans, ws, ys):
        p.conv2d(x, w, y)
        x = y
    return x


def work(case):
    """The first x, every w and the last y once; the multiplications and additions of the
    Winograd-domain channel sums."""
    layers = _layers(case)
    out = layers[-1]
    values = case["B"] * layers[0]["M"] * case["H"] * case["W"] + math.prod(_out_shape(out))
    flops = 0.0
    for s in layers:
        values += s["N"] * (1 if s["depthwise"] else s["M"]) * s["r"] * s["r"]
        g = _geometry(s)
        flops += 2.0 * g["ewmm_mults"] if s["depthwise"] else g["contract_flop"]
    return {"bytes": 4.0 * values, "flops": flops}


def tolerance(case):
    """About four times the error against 64 bits that is measured (the largest over the listed
    cases and forty drawn ones), by what sets it: the nest's bases and depth (each level's
    transforms add to it), the channels summed, or the 16-bit pairs of the split."""
    if case["kind"] == "stack":
        return {"rel": 1e-5}
    g = _geometry(case)
    if case["split"]:
        return {"rel": {1: 2.5e-5, 2: 4e-5, 3: 6e-5, 4: 1e-4}[g["n"]]}
    if g["tile"] == nwg.NWG_TILE_F3X3_3X3:
        return {"rel": {0: 2e-6, 1: 4e-6, 2: 3e-5}[g["n"]]}
    if g["tile"] == nwg.NWG_TILE_MIX_F23_F33:
        return {"rel": 1.5e-5 if g["n"] == 3 else 5e-5}
    if case["depthwise"]:
        return {"rel": {0: 1e-6, 1: 1e-6, 2: 1e-6, 3: 1.5e-6, 4: 2.2e-6}[g["n"]]}
    return {"rel": {0: 2e-6, 1: 2e-6, 2: 2e-6, 3: 4.5e-6, 4: 6e-6}[g["n"]]}


def _exact_layer(x, w, pad, depthwise):
    """Direct correlation in 64 bits, one tap at a time."""
    B, M, H, W = x.shape
    N, r = w.shape[0], w.shape[2]
    Ho, Wo = H + 2 * pad - r + 1, W + 2 * pad - r + 1
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    if depthwise:
        y = torch.zeros((B, N, Ho, Wo), dtype=torch.float64, device=x.device)
        for u in range(r):
            for v in range(r):
                y += xp[:, :, u:u + Ho, v:v + Wo] * w[:, 0, u, v].reshape(1, N, 1, 1)
        return y
    xp = xp.transpose(0, 1).contiguous()            # [M][B][rows][columns]
    y = torch.zeros((N, B * Ho * Wo), dtype=torch.float64, device=x.device)
    for u in range(r):
        for v in range(r):
            y += w[:, :, u, v].contiguous() @ xp[:, :, u:u + Ho, v:v + Wo].reshape(M, -1)
    return y.reshape(N, B, Ho, Wo).transpose(0, 1).contiguous()


def exact(case, seed):
    x, ws = _inputs(case, seed)
    x = x.double()
    for s, w in zip(_layers(case), ws):
        x = _exact_layer(x, w.double(), s["pad"], s["depthwise"])
    return x
