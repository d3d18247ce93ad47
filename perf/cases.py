"""Workloads that stand for the use of this framework, for timing and for comparing outputs.

A case is a dict of plain values.  listed() names the standing ones, draw() gives more of the same ranges, prepare() makes
what a program has in hand before the call, run() is one pass through the public entry points, work() the bytes and
operations that pass cannot do without, tolerance() how far another correct implementation may be off.

Kinds of cases
  block    one dynamic bottleneck, out of place (the caller keeps its input): patch mask given from outside, or decided by the
           spatial masker (fused into the first 1x1 below S = 7, a call of its own from S = 7 on)
  stage    one stage of a backbone: first block (static or dynamic, projection shortcut) into a new map, then dynamic
           identity blocks in place, each with its own masker and, optionally, a keep gate per sample
  channel  channel masker + channel-skipping bottleneck at the four ResNet stages
  body     a whole ResNet-50 / -101 from the image, patch masks or layer gates from outside
  regnety  a whole RegNetY from the image (group convolution + SE blocks), patch masks or layer gates from outside

Shapes: ResNet-50 / -101 and RegNetY-400MF / -800MF at 224 x 224 and other image sizes, granularity 4-4-2-1.  Activations
behind a ReLU, Kaiming-normal weights, folded-BN affines near one; active patches form coherent regions, as a trained masker
selects them, and stand out in the features (a masker separates them clearly, so rounding does not move a decision).
"""
from __future__ import annotations

import math

import torch

import paper_2308_15949_amd as L
from paper_2308_15949_amd import binding as B
from paper_2308_15949_amd import inputs as I

GRANULARITY = (4, 4, 2, 1)
DEPTHS = {"resnet50": (3, 4, 6, 3), "resnet101": (3, 4, 23, 3), "regnety400": (1, 3, 6, 6), "regnety800": (1, 3, 8, 2)}
REGNETY = {"regnety400": "400MF", "regnety800": "800MF"}
COHERENT_BLUR = 3  # window of the box blur that makes active regions coherent


# ----- cases ------------------------------------------------------------------------------------------------------------
def listed() -> list[dict]:
    return [
        # one float32 image through one stage-1 block, mask from outside: the smallest call (latency, launches)
        dict(name="block1_f32_b1", kind="block", model="resnet50", stage=1, n=1, h=224, w=224, dtype="f32", S=4, ratio=0.5,
             mask="given"),
        # the headline workload: the stage-3 block with its masker, a server batch
        dict(name="block3_b128", kind="block", model="resnet101", stage=3, n=128, h=224, w=224, dtype="bf16", S=2, ratio=0.5,
             mask="masker"),
        # stage by stage as a model runs them: wide maps with few channels ...
        dict(name="stage1_b128", kind="stage", model="resnet50", stage=1, n=128, h=224, w=224, dtype="bf16", S=4, ratio=0.5,
             first="static", keep=1.0),
        # ... an odd batch of non-square images with coarse patches and a dynamic first block ...
        dict(name="stage2_b27_coarse", kind="stage", model="resnet50", stage=2, n=27, h=224, w=336, dtype="bf16", S=7,
             ratio=0.4, first="dynamic", keep=1.0),
        # ... a single image: serving, latency-bound ...
        dict(name="stage3_b1", kind="stage", model="resnet50", stage=3, n=1, h=224, w=224, dtype="bf16", S=2, ratio=0.5,
             first="static", keep=1.0),
        # ... small maps with many channels
        dict(name="stage4_b128", kind="stage", model="resnet50", stage=4, n=128, h=224, w=224, dtype="bf16", S=1, ratio=0.5,
             first="static", keep=1.0),
        # channel skipping with its masker, four groups, at all four stages
        dict(name="channel_b64", kind="channel", n=64, h=224, w=224, dtype="bf16", D=4),
        # whole models: a single image, a server batch with patch masks, a larger one with layer skipping
        dict(name="resnet50_b1", kind="body", model="resnet50", n=1, h=224, w=224, dtype="bf16", skip="spatial", ratio=0.5),
        dict(name="resnet101_b128", kind="body", model="resnet101", n=128, h=224, w=224, dtype="bf16", skip="spatial",
             ratio=0.5),
        dict(name="resnet101_b256_layer", kind="body", model="resnet101", n=256, h=224, w=224, dtype="bf16", skip="layer",
             ratio=0.6),
        # the lightweight backbones: one stage with maskers, a whole model with layer skipping
        dict(name="regnety400_stage3_b32", kind="stage", model="regnety400", stage=3, n=32, h=224, w=224, dtype="bf16", S=2,
             ratio=0.5, first="static", keep=1.0),
        dict(name="regnety800_b128_layer", kind="regnety", model="regnety800", n=128, h=224, w=224, dtype="bf16",
             skip="layer", ratio=0.6),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng) -> dict:
    kind = rng.choice(("block", "block", "stage", "stage", "stage", "channel", "body", "body", "regnety"))
    h, w = 32 * rng.randint(5, 9), 32 * rng.randint(5, 9)
    if rng.random() < 0.5:
        h = w = 224
    area = h * w / (224 * 224)
    n = _log_int(rng, 1, max(1, int(128 / area)))
    ratio = round(rng.uniform(0.15, 0.9), 3)
    c = dict(kind=kind, n=n, h=h, w=w, dtype="bf16")
    if kind in ("block", "stage"):
        c["model"] = rng.choice(("resnet50", "resnet101") if kind == "block" else ("resnet50", "resnet50", "regnety400", "regnety800"))
        c["stage"] = s = rng.randint(1, 4)
        down, usual = 2 ** (s + 1), GRANULARITY[s - 1]
        # from one pixel per patch (narrow maps in a chain: from the usual granularity) to about twice the usual granularity
        low = 1 if kind == "block" or (s == 3 and c["model"] not in REGNETY) else usual if c["model"] in REGNETY else (usual + 1) // 2
        c["S"] = rng.choice([v for v in (1, 2, 4, 7, 8) if low <= v <= 2 * usual + 3 and v < h // down
                             and (h // down) % v == 0 and (w // down) % v == 0])
        c["ratio"] = ratio
        if rng.random() < 0.2:
            c["dtype"], c["n"] = "f32", min(n, 32)
    if kind == "block":
        c["mask"] = rng.choice(("given", "masker", "masker"))
    elif kind == "stage":
        c["first"] = rng.choice(("static", "dynamic"))
        c["keep"] = 0.6 if c["n"] > 7 and rng.random() < 0.3 else 1.0
    elif kind == "channel":
        c["D"] = rng.choice((2, 4, 4, 4, 8))
        c["n"] = min(n, max(1, int(64 / area)))
    else:
        c["model"] = rng.choice(("resnet50", "resnet101") if kind == "body" else ("regnety400", "regnety800"))
        c["skip"] = rng.choice(("spatial", "layer"))
        c["ratio"] = ratio
    return c


# ----- shapes -----------------------------------------------------------------------------------------------------------
def _stage_shape(model: str, stage: int) -> tuple[int, int, int, int, int | None]:
    """(channels before the stage, mid, out, stride of the first block, group width or None)."""
    if model in REGNETY:
        cfg = I.REGNETY[REGNETY[model]]
        c = cfg["stages"][stage]["c"]
        return (32 if stage == 1 else cfg["stages"][stage - 1]["c"]), c, c, 2, cfg["g"]
    m = I.STAGES[stage]["m"]
    return (64 if stage == 1 else 2 * m), m, 4 * m, (1 if stage == 1 else 2), None


def _map(case: dict, stage: int) -> tuple[int, int]:
    """Height and width of a stage's feature maps."""
    d = 2 ** (stage + 1)
    return case["h"] // d, case["w"] // d


# ----- what a program holds -----------------------------------------------------------------------------------------------
class _Maker:
    """Draws tensors from one seeded generator on the GPU and keeps them alive."""

    def __init__(self, case: dict, seed: int):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.bf16 = case["dtype"] == "bf16"
        self.dt = torch.bfloat16 if self.bf16 else torch.float32
        self.code = B.BF16 if self.bf16 else B.F32
        self.held = []

    def keep(self, t):
        self.held.append(t)
        return t

    def randn(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def weight(self, *shape, fan_in: int):
        return self.keep((self.randn(*shape) * math.sqrt(2.0 / fan_in)).to(self.dt))

    def affine(self, c: int, gain: float = 1.0):
        return self.keep(gain * (1.0 + 0.1 * self.randn(c))), self.keep(0.1 * self.randn(c))

    def empty(self, *shape, dtype=None):
        return self.keep(torch.empty(shape, dtype=dtype or self.dt, device="cuda"))

    def workspace(self, nbytes: int):
        return self.empty(max(int(nbytes), 256), dtype=torch.uint8)

    def block(self, c_in: int, m: int, c_out: int, gain: float, gw: int | None = None):
        """Descriptor of a bottleneck; weights laid out once, as at model load."""
        w1 = self.weight(m, c_in, fan_in=c_in)
        w2 = self.weight(m, 3, 3, gw or m, fan_in=9 * (gw or m))
        w3 = self.weight(c_out, m, fan_in=m)
        d = L.make_bottleneck(w1, w2, w3, *self.affine(m), *self.affine(m), *self.affine(c_out, gain), True)
        nb = L.packed_weights_size(d, self.code) if gw is None else 0
        if nb:
            packed = self.empty(nb, dtype=torch.uint8)
            L.laud_pack_weights(d, self.code, packed)
            d.packed = packed.data_ptr()
        return self.keep(d)

    def se(self, c: int, width: int, gw: int):
        t = [self.keep(v) for v in (self.randn(width, c) * math.sqrt(2.0 / c), 0.1 * self.randn(width),
                                    self.randn(c, width) * math.sqrt(4.0 / width), 0.5 * self.randn(c))]
        return self.keep(L.make_group_se(gw, *t))

    def shortcut(self, c_in: int, c_out: int):
        return (self.weight(c_out, c_in, fan_in=c_in), *self.affine(c_out, 0.5))

    def regions(self, n: int, hp: int, wp: int, ratio: float):
        """Coherent patch mask [n, hp, wp] (bool) with round(ratio * patches) active patches over the batch."""
        f = torch.nn.functional.avg_pool2d(self.randn(n, 1, hp + 2, wp + 2), COHERENT_BLUR, 1).reshape(-1)
        k = min(max(int(round(ratio * f.numel())), 1), max(f.numel() - 1, 1))
        mask = torch.zeros(f.numel(), dtype=torch.bool, device="cuda")
        mask[f.topk(k).indices] = True
        return mask.view(n, hp, wp)

    def gates(self, n: int, p: float):
        return torch.rand(n, generator=self.g, device="cuda") < p

    def features(self, n: int, h: int, w: int, c: int, regions=None):
        """Activations behind a ReLU; larger inside the active regions."""
        x = self.randn(n, h, w, c)
        if regions is not None:
            up = regions.repeat_interleave(h // regions.shape[1], 1).repeat_interleave(w // regions.shape[2], 2)
            x += 1.5 * up.unsqueeze(-1)
        return self.keep(x.relu_().to(self.dt))

    def masker(self, x, S: int, regions):
        """Masker weights and bias that separate the regions of x, as training would leave them."""
        n, h, w, c = x.shape
        p = x.float().view(n, h // S, S, w // S, S, c).mean((2, 4)).reshape(-1, c)
        on = regions.reshape(-1)
        d = p[on].mean(0) - p[~on].mean(0)
        d /= d.norm()
        logit = (p * d).sum(1)
        return self.keep(d.contiguous()), -0.5 * float(logit[on].min() + logit[~on].max())

    def lists(self, n: int):
        return (self.keep(torch.zeros(n, dtype=torch.uint8, device="cuda")), self.keep(torch.zeros(n, dtype=torch.int32, device="cuda")),
                self.keep(torch.zeros(1, dtype=torch.int32, device="cuda")))


def _prepare_block(mk: _Maker, case: dict) -> dict:
    _, m, c, _, _ = _stage_shape(case["model"], case["stage"])
    h, w = _map(case, case["stage"])
    n, S = case["n"], case["S"]
    on = mk.regions(n, h // S, w // S, case["ratio"])
    x = mk.features(n, h, w, c, on)
    out, fx, p = mk.empty(n, h, w, c), L.fmap_of(x), mk.block(c, m, c, 1.0)
    mask, idx, count = mk.lists(on.numel())
    ws = mk.workspace(L.workspace_size(B.OP_DYN_BOTTLENECK, fx, p, S))
    if case["mask"] == "given":
        mask.copy_(on.reshape(-1))
        wc = mk.workspace(L.workspace_size(B.OP_COMPACT, fx, None, on.numel()))
        ops = [(L.laud_layer_skip_compact, (mask, on.numel(), idx, count, wc)),
               (L.laud_dyn_bottleneck, (x, fx, p, S, idx, count, out, ws))]
    else:
        wm, bias = mk.masker(x, S, on)
        if S < 7:
            ops = [(L.laud_masker_dyn_bottleneck, (x, fx, p, S, wm, bias, None, mask, idx, count, None, None, out, ws))]
        else:
            wsm = mk.workspace(L.workspace_size(B.OP_MASK_GEN, fx, None, S))
            ops = [(L.laud_mask_gen, (x, fx, S, wm, bias, None, mask, idx, count, None, None, wsm)),
                   (L.laud_dyn_bottleneck, (x, fx, p, S, idx, count, out, ws))]
    return {"ops": ops, "out": (out, mask, idx, count)}


def _play(ops) -> None:
    for fn, args in ops:
        fn(*args)


def _prepare_stage(mk: _Maker, case: dict) -> dict:
    c_in, m, c, stride, gw = _stage_shape(case["model"], case["stage"])
    h, w = _map(case, case["stage"])
    n, S = case["n"], case["S"]
    se = gw is not None
    on = mk.regions(n, h // S, w // S, case["ratio"])
    xin = mk.features(n, h * stride, w * stride, c_in, on)
    fin, x = L.fmap_of(xin), mk.empty(n, h, w, c)
    fx = L.fmap_of(x)
    mask, idx, count = mk.lists(on.numel())
    # the first block writes the stage's map
    p, sc = mk.block(c_in, m, c, 0.5, gw), mk.shortcut(c_in, c)
    e = mk.se(m, max(8, c_in // 4), gw) if se else None
    ops = []
    if case["first"] == "dynamic":
        wm, bias = mk.masker(xin, stride * S, on)
        wsm = mk.workspace(L.workspace_size(B.OP_MASK_GEN, fin, None, stride * S))
        ops.append((L.laud_mask_gen, (xin, fin, stride * S, wm, bias, None, mask, idx, count, None, None, wsm)))
        first_idx, first_count = idx, count
    elif se:  # the static first block of these backbones: every patch of the output grid listed
        first_idx = mk.keep(torch.arange(on.numel(), dtype=torch.int32, device="cuda"))
        first_count = mk.keep(torch.full((1,), on.numel(), dtype=torch.int32, device="cuda"))
    if se or case["first"] == "dynamic":
        wsp = mk.workspace(L.dyn_projection_workspace(fin, p, stride))
        if se:
            ops.append((L.laud_dyn_group_se_projection_bottleneck, (xin, fin, p, e, *sc, stride, S, first_idx, first_count, x, wsp)))
        else:
            ops.append((L.laud_dyn_projection_bottleneck, (xin, fin, p, *sc, stride, S, first_idx, first_count, x, wsp)))
    else:
        wsp = mk.workspace(L.static_bottleneck_workspace(fin, p, stride))
        ops.append((L.laud_static_bottleneck, (xin, fin, p, *sc, stride, x, wsp)))
    _play(ops)
    # identity blocks in place, every one with a masker fitted to the features it meets
    ws = wsm = None
    for _ in range(DEPTHS[case["model"]][case["stage"] - 1] - 1 or 1):
        p = mk.block(c, m, c, 0.25, gw)
        e = mk.se(m, max(8, c // 4), gw) if se else None
        keep = None
        if case["keep"] < 1.0:
            keep = mk.keep(mk.gates(n, case["keep"]).to(torch.uint8))
        if ws is None:
            ws = mk.workspace(L.workspace_size(B.OP_DYN_BOTTLENECK, fx, p, S))
            wsm = mk.workspace(L.workspace_size(B.OP_MASK_GEN, fx, None, S))
        wm, bias = mk.masker(x, S, on)
        if se:
            step = [(L.laud_mask_gen, (x, fx, S, wm, bias, keep, mask, idx, count, None, None, wsm)),
                    (L.laud_dyn_group_se_bottleneck, (x, fx, p, e, S, idx, count, x, ws))]
        elif S < 7:
            step = [(L.laud_masker_dyn_bottleneck, (x, fx, p, S, wm, bias, keep, mask, idx, count, None, None, x, ws))]
        else:
            step = [(L.laud_mask_gen, (x, fx, S, wm, bias, keep, mask, idx, count, None, None, wsm)),
                    (L.laud_dyn_bottleneck, (x, fx, p, S, idx, count, x, ws))]
        _play(step)
        ops += step
    return {"ops": ops, "out": (x, mask, count)}


def _prepare_channel(mk: _Maker, case: dict) -> dict:
    ops, out, n, D = [], [], case["n"], case["D"]
    for stage in (1, 2, 3, 4):
        _, m, c, _, _ = _stage_shape("resnet50", stage)
        h, w = _map(case, stage)
        # channels differ in strength from sample to sample: that is what the masker sees
        x = mk.keep((mk.randn(n, h, w, c) + mk.randn(n, 1, 1, c)).relu_().to(mk.dt))
        y, fx, p = mk.empty(n, h, w, c), L.fmap_of(x), mk.block(c, m, c, 0.25)
        hidden = max(D // 16, 16)
        wa, ba = mk.keep(mk.randn(hidden, c) * math.sqrt(2.0 / c)), mk.keep(0.1 * mk.randn(hidden))
        wb, bb = mk.keep(mk.randn(2 * D, hidden) / math.sqrt(hidden)), mk.keep(0.1 * mk.randn(2 * D))
        cmask = mk.keep(torch.zeros((n, D), dtype=torch.uint8, device="cuda"))
        wsm = mk.workspace(L.channel_masker_workspace(fx))
        ws = mk.workspace(L.workspace_size(B.OP_CHANNEL_SKIP, fx, p, D))
        ops += [(L.laud_channel_masker, (x, fx, wa, ba, hidden, wb, bb, D, cmask, None, wsm)),
                (L.laud_channel_skip_conv, (x, fx, p, cmask, D, y, ws))]
        out += [y, cmask]
    return {"ops": ops, "out": tuple(out)}


def _prepare_body(mk: _Maker, case: dict) -> dict:
    n, h, w, model = case["n"], case["h"], case["w"], case["model"]
    se = model in REGNETY
    img = mk.keep(mk.randn(n, h, w, 3).to(mk.dt))
    if se:
        c0, x = 32, mk.empty(n, h // 2, w // 2, 32)
        ops = [(L.laud_stem3x3, (img, n, h, w, mk.code, mk.weight(32, 3, 3, 3, fan_in=27), *mk.affine(32), 32, x))]
    else:
        c0, x = 64, mk.empty(n, h // 4, w // 4, 64)
        ops = [(L.laud_stem, (img, n, h, w, mk.code, mk.weight(64, 7, 7, 3, fan_in=147), *mk.affine(64), 64, x,
                              mk.workspace(L.stem_workspace(n, h, w, 64, mk.code))))]
    maps = []  # every stage's map: what a classifier, or a detector's neck, goes on from
    for stage, depth in enumerate(DEPTHS[model], 1):
        c_in, m, c, stride, gw = _stage_shape(model, stage)
        hs, ws_ = _map(case, stage)
        fin, y = L.fmap_of(x), mk.empty(n, hs, ws_, c)
        p, sc = mk.block(c_in, m, c, 0.5, gw), mk.shortcut(c_in, c)
        S = GRANULARITY[stage - 1]
        if se:
            every = n * (hs // S) * (ws_ // S)
            ids = mk.keep(torch.arange(every, dtype=torch.int32, device="cuda"))
            cnt = mk.keep(torch.full((1,), every, dtype=torch.int32, device="cuda"))
            ops.append((L.laud_dyn_group_se_projection_bottleneck, (
                x, fin, p, mk.se(m, max(8, c_in // 4), gw), *sc, stride, S, ids, cnt, y,
                mk.workspace(L.dyn_projection_workspace(fin, p, stride)))))
        else:
            ops.append((L.laud_static_bottleneck, (x, fin, p, *sc, stride, y,
                                                   mk.workspace(L.static_bottleneck_workspace(fin, p, stride)))))
        x, fx, ws = y, L.fmap_of(y), None
        maps.append(y)
        for _ in range(depth - 1):
            p = mk.block(c, m, c, 0.25, gw)
            if case["skip"] == "layer":
                keep = mk.gates(n, case["ratio"])
                if stage == 3 and not se:  # the gate combined with a patch mask
                    given, Sb = keep.view(n, 1, 1) & mk.regions(n, hs // S, ws_ // S, 0.5), S
                elif hs == ws_:
                    given, Sb = keep, hs
                else:  # patches are square: a kept sample lists all of its patches
                    given, Sb = keep.view(n, 1, 1).expand(n, hs // S, ws_ // S), S
            else:
                given, Sb = mk.regions(n, hs // S, ws_ // S, case["ratio"]), S
            given = mk.keep(given.reshape(-1).to(torch.uint8))
            _, idx, cnt = mk.lists(given.numel())
            wc = mk.workspace(L.workspace_size(B.OP_COMPACT, fx, None, given.numel()))
            if ws is None:
                ws = mk.workspace(L.workspace_size(B.OP_DYN_BOTTLENECK, fx, p, S))
            ops.append((L.laud_layer_skip_compact, (given, given.numel(), idx, cnt, wc)))
            if se:
                ops.append((L.laud_dyn_group_se_bottleneck, (x, fx, p, mk.se(m, max(8, c // 4), gw), Sb, idx, cnt, x, ws)))
            else:
                ops.append((L.laud_dyn_bottleneck, (x, fx, p, Sb, idx, cnt, x, ws)))
    return {"ops": ops, "out": tuple(maps)}


def prepare(case: dict, seed: int) -> dict:
    mk = _Maker(case, seed)
    make = {"block": _prepare_block, "stage": _prepare_stage, "channel": _prepare_channel}.get(case["kind"], _prepare_body)
    state = make(mk, case)
    state["held"] = mk.held
    return state


def run(state: dict):
    for fn, args in state["ops"]:
        fn(*args)
    return state["out"]


# ----- what a pass cannot do without ------------------------------------------------------------------------------------
def _block_work(case, n, h, w, c_in, m, c_out, gw, ratio, reads, writes, out_hw=None):
    """Bytes and operations of one block at an activation ratio; reads / writes: shares of its maps that move."""
    eb = 2 if case["dtype"] == "bf16" else 4
    ho, wo = out_hw or (h, w)
    wts = (c_in * m + 9 * m * (gw or m) + m * c_out + (c_in * c_out if out_hw else 0)) * eb
    flops = 2.0 * n * ho * wo * (ratio * (c_in * m + 9 * m * (gw or m) + m * c_out) + (c_in * c_out if out_hw else 0))
    return n * h * w * c_in * eb * reads + n * ho * wo * c_out * eb * writes + wts, flops


def work(case: dict) -> dict:
    n, kind, parts = case["n"], case["kind"], []
    if kind == "block":
        _, m, c, _, _ = _stage_shape(case["model"], case["stage"])
        parts.append(_block_work(case, n, *_map(case, case["stage"]), c, m, c, None, case["ratio"], 1.0, 1.0))
    elif kind == "channel":
        for stage in (1, 2, 3, 4):
            _, m, c, _, _ = _stage_shape("resnet50", stage)
            h, w = _map(case, stage)
            b, _ = _block_work(case, n, h, w, c, m, c, None, 1.0, 1.0, 1.0)
            parts.append((b, 2.0 * n * h * w * (0.5 * 2 * c * m + 0.25 * 9 * m * m)))  # half of the groups kept
    else:
        stages = [case["stage"]] if kind == "stage" else [1, 2, 3, 4]
        for stage in stages:
            c_in, m, c, stride, gw = _stage_shape(case["model"], stage)
            h, w = _map(case, stage)
            first = case["ratio"] if case.get("first") == "dynamic" else 1.0
            parts.append(_block_work(case, n, h * stride, w * stride, c_in, m, c, gw, first, 1.0, 1.0, (h, w)))
            r = case["ratio"] * case.get("keep", 1.0)
            if case.get("skip") == "layer" and stage == 3 and kind == "body":
                r *= 0.5
            depth = DEPTHS[case["model"]][stage - 1] - 1
            # a masker reads its whole map, a block with given patches only those; only the active patches are written
            reads = 1.0 if kind == "stage" else r
            parts += [_block_work(case, n, h, w, c, m, c, gw, r, reads, r)] * (max(depth, 1) if kind == "stage" else depth)
        if kind != "stage":
            eb, h, w = 2, case["h"], case["w"]
            c0, k, d = (32, 27, 2) if kind == "regnety" else (64, 147, 4)
            parts.append((n * h * w * 3 * eb + n * (h // d) * (w // d) * c0 * eb, 2.0 * n * (h // 2) * (w // 2) * c0 * k))
    return {"bytes": float(sum(b for b, _ in parts)), "flops": float(sum(f for _, f in parts))}


def tolerance(case: dict):
    """float32: sums of up to a few thousand products.  bf16: intermediates rounded to eight bits once per convolution;
    a chain of blocks carries the differences on."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5 if case["kind"] == "block" else 3e-5, "max": 1e-3}
    if case["kind"] in ("block", "channel"):
        return {"rel": 1e-2, "max": 0.2}
    return {"rel": 2e-2, "max": 0.5}
