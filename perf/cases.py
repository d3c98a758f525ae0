"""Timed cases of the library, through its Python binding.

What a program that uses the library spends its GPU time on: filtering a frame
(``Context.filter``) with a procedural, stored or learned texture, filtering a
stack of material layers (``Context.filter_layers``), producing raw texels
(``Texture.eval``), and fitting a learned texture (``Decoder.loss_grad``,
``Decoder.train``).  Frames are perspective views of a few seeded textured
planes, scaled so that a given share of the pixels magnifies, as in the
repository's benchmark; everything is drawn from the seed on the GPU.

``exact`` computes the same results in float64 with plain torch: the texel
lattice, the discrete decisions (float32, the op order the library documents)
and the weighting.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2506_17770_amd as ctf

KIND = {"bilinear4": ctf.BILINEAR4, "stf1": ctf.STF1, "list": ctf.LIST, "box": ctf.BOX, "mask": ctf.MASK}
FILTER = {"bilinear": ctf.FILTER_BILINEAR, "bspline": ctf.FILTER_BSPLINE, "catmull_rom": ctf.FILTER_CATMULL_ROM}
FALLBACK = {"stf1": ctf.FB_STF1, "c": ctf.FB_C, "cplus": ctf.FB_CPLUS}
WAVE = {"8x8": ctf.WAVE_8X8, "8x4": ctf.WAVE_8X4}
PREC = {"fp16": ctf.FP16, "bf16": ctf.BF16}

HIDDEN, CHANNELS = 64, 8
MLP_FLOP = 2 * (16 * 64 + 64 * 64 + 64 * 4)   # one decoded texel
TERM_FLOP = 8                                 # phase (2 FMA), fract, sine, accumulate


def _frame(name, tex, w, h, method, **more):
    c = dict(op="filter", tex=tex, width=w, height=h, method=method, k=1, box=0, filter="bilinear",
             fallback="stf1", wave="8x8", tex_w=2048, terms=32, l0=512, l1=128, precision="fp16",
             planes=4, magnify=0.7)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # an icon-sized view of a small material: launch-bound
        _frame("tiny_256_list", "sinusoids", 256, 256, "list", tex_w=64, terms=8, planes=1, magnify=0.9),
        # a full-HD frame with a costly procedural material: the exact
        # duplicate-free set, the full filter it replaces, and the paper's
        # 32-lane waves with its best fallback
        _frame("proc_1080p_list", "sinusoids", 1920, 1080, "list"),
        _frame("proc_1080p_bilinear4", "sinusoids", 1920, 1080, "bilinear4"),
        _frame("proc_1080p_mask_cplus_8x4", "sinusoids", 1920, 1080, "mask", fallback="cplus", wave="8x4"),
        # a window of odd size, learned texture in bf16, one texel per lane
        _frame("dec_ragged_mask_bf16", "decoder", 1279, 717, "mask", precision="bf16"),
        # a 4K frame of a learned texture: collaborative, the full filter, and
        # the smooth (cubic) filter
        _frame("dec_4k_list_fp16", "decoder", 3840, 2160, "list", k=4),
        _frame("dec_4k_bilinear4_fp16", "decoder", 3840, 2160, "bilinear4"),
        _frame("dec_4k_bspline_list_fp16", "decoder", 3840, 2160, "list", k=4, filter="bspline"),
        # a 4K frame of a six-layer material (albedo, normal, roughness ...)
        dict(name="layers_4k_list_fp16", op="layers", layers=6, width=3840, height=2160, method="list", k=4,
             filter="bilinear", tex_w=2048, l0=512, l1=128, precision="fp16", planes=4, magnify=0.7),
        # fitting: the gradient of one batch (forward and backward), and a
        # stretch of training up to reading the weights back
        dict(name="loss_grad_65536_bf16", op="loss_grad", batch=65536, tex_w=2048, terms=32, l0=512, l1=128,
             precision="bf16"),
        dict(name="train_200_65536_bf16", op="train", steps=200, batch=65536, tex_w=2048, terms=32, l0=512, l1=128,
             precision="bf16"),
        # expanding a learned texture to all its texels
        dict(name="eval_2048_fp16", op="eval", tex="decoder", texels=2048 * 2048, tex_w=2048, terms=32, l0=512,
             l1=128, precision="fp16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["filter", "filter", "filter", "filter", "filter", "filter", "layers", "loss_grad", "train",
                     "eval"])
    l0 = rng.choice([128, 256, 512])
    dec = dict(tex_w=2048, l0=l0, l1=l0 // 4, precision=rng.choice(["fp16", "bf16"]))
    if op == "filter":
        w = _log_int(rng, 203, 3840)
        h = max(77, min(2160, int(w * rng.uniform(0.4, 0.7))))
        tex = rng.choice(["sinusoids", "sinusoids", "decoder", "decoder", "decoder", "table"])
        method = rng.choice(["list", "list", "mask", "mask", "box", "bilinear4", "stf1"])
        c = _frame(None, tex, w, h, method, planes=rng.randint(1, 4), magnify=round(rng.uniform(0.3, 1.0), 3), **dec)
        c["k"] = rng.choice([1, 1, 2, 4, 4])
        c["box"] = rng.choice([0, 4, 6])
        if tex == "sinusoids":
            c.update(tex_w=rng.choice([64, 512, 2048, 4096]), terms=rng.choice([8, 13, 32, 48]))
        if tex == "table":
            c["tex_w"] = rng.choice([256, 1024, 2048])
        if tex != "decoder" and rng.random() < 0.3:
            c["wave"] = "8x4"
        # the 16-tap full filter of a whole 4K frame would cost more than the
        # largest listed case
        if rng.random() < 0.25 and method != "bilinear4":
            c["filter"] = rng.choice(["bspline", "catmull_rom"])
        if method in ("list", "mask", "box") and rng.random() < 0.2:
            c["fallback"] = rng.choice(["c", "cplus"])
        return c
    if op == "layers":
        w = _log_int(rng, 320, 3840)
        return dict(op="layers", layers=rng.randint(2, 6), width=w, height=max(77, min(2160, int(w * 0.5625))),
                    method=rng.choice(["list", "mask"]), k=rng.choice([1, 4]), filter="bilinear",
                    planes=rng.randint(1, 4), magnify=round(rng.uniform(0.3, 1.0), 3), **dec)
    if op == "loss_grad":
        return dict(op="loss_grad", batch=_log_int(rng, 1000, 65536), terms=32, **dec)
    if op == "train":
        return dict(op="train", steps=rng.randint(20, 200), batch=_log_int(rng, 1000, 65536), terms=32, **dec)
    tex = rng.choice(["decoder", "decoder", "sinusoids"])
    return dict(op="eval", tex=tex, texels=_log_int(rng, 1000, 2048 * 2048), terms=rng.choice([8, 32]), **dec)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed, what):
    """numpy generator of one kind of input."""
    return np.random.default_rng([int(seed), what])


def _terms(case, seed):
    """(p, q, j) and amplitudes of the procedural texture."""
    rng, K, W = _gen(seed, 1), case["terms"], case["tex_w"]
    F = max(1, min(64, W // 8))
    pqj = np.empty((4, K, 3), np.int32)
    pqj[..., 0] = rng.integers(1, F + 1, (4, K)) * rng.choice([-1, 1], (4, K))
    pqj[..., 1] = rng.integers(-F, F + 1, (4, K))
    pqj[..., 2] = rng.integers(0, W, (4, K))
    amp = rng.uniform(0.5, 1.5, (4, K))
    return pqj, (amp / amp.sum(1, keepdims=True)).astype(np.float32)


def _params(case, seed):
    """Flat decoder parameters: latents of a fitted texture's size, He-uniform
    weights, small biases (a fresh decoder's latents for fitting)."""
    rng, l0, l1, H = _gen(seed, 2), case["l0"], case["l1"], HIDDEN
    lat = 0.5 if case["op"] in ("filter", "layers", "eval") else 1e-2
    u = lambda n, a: rng.uniform(-a, a, n)  # noqa: E731
    p = [u((l0 * l0 + l1 * l1) * CHANNELS, lat), u(16 * H, math.sqrt(6 / 16)), u(H, 0.1),
         u(H * H, math.sqrt(6 / H)), u(H, 0.1), u(H * 4, math.sqrt(6 / H)), np.full(4, 0.5)]
    return np.concatenate(p).astype(np.float32)


def _table(case, seed):
    g = torch.Generator().manual_seed(int(seed) * 7 + 3)
    return torch.rand((case["tex_w"], case["tex_w"], 4), generator=g, dtype=torch.float32).numpy()


def _scene(case, seed):
    """uv [H][W][2] and derivatives [H][W][4] of the nearest of a few random
    planes under a 60 degree camera; the world is scaled so that a share
    ``magnify`` of the visible pixels has at most one texel per pixel."""
    w, h, rng = case["width"], case["height"], _gen(seed, 3)
    f64 = dict(dtype=torch.float64, device="cuda")
    th = math.tan(math.radians(30.0))
    x = ((2 * (torch.arange(w, **f64) + 0.5) / w - 1) * th * w / h)[None, :].expand(h, w)
    y = ((1 - 2 * (torch.arange(h, **f64) + 0.5) / h) * th)[:, None].expand(h, w)
    step = (2 * th / h, -2 * th / h)          # d(ray x)/dpx, d(ray y)/dpy; ray z = -1
    near = torch.full((h, w), math.inf, **f64)
    uv = torch.full((h, w, 2), math.nan, **f64)
    duv = torch.full((h, w, 4), math.nan, **f64)
    for _ in range(case["planes"]):
        cz = rng.uniform(math.cos(math.radians(75)), 1.0)
        az, sz, phi = rng.uniform(0, 2 * math.pi), math.sqrt(1 - cz * cz), rng.uniform(0, 2 * math.pi)
        n = np.array([sz * math.cos(az), sz * math.sin(az), cz])
        a = np.cross(n, [1.0, 0, 0] if abs(n[0]) < 0.9 else [0, 1.0, 0])
        a /= np.linalg.norm(a)
        e1 = math.cos(phi) * a + math.sin(phi) * np.cross(n, a)
        e2 = np.cross(n, e1)
        depth = rng.uniform(1.0, 4.0)
        o = np.array([*(rng.uniform(-0.6, 0.6, 2) * depth), -depth])
        size = math.exp(rng.uniform(math.log(0.5), math.log(2.0)))
        off = rng.uniform(0, 1, 2)
        dn, on = x * n[0] + y * n[1] - n[2], float(o @ n)
        lam = on / dn
        take = torch.isfinite(lam) & (lam > 0) & (lam < near)
        near = torch.where(take, lam, near)
        got, dgot = [], [[], []]
        for e, f in ((e1, off[0]), (e2, off[1])):
            ray = x * e[0] + y * e[1] - e[2]
            got.append((lam * ray - float(o @ e)) / size + f)
            for ax in range(2):
                dgot[ax].append((-on * step[ax] * n[ax] / (dn * dn) * ray + lam * step[ax] * e[ax]) / size)
        uv = torch.where(take[..., None], torch.stack(got, -1), uv)
        duv = torch.where(take[..., None], torch.stack(dgot[0] + dgot[1], -1), duv)
    d = duv * case["tex_w"]
    ratio = torch.sqrt(torch.maximum(d[..., 0] ** 2 + d[..., 1] ** 2, d[..., 2] ** 2 + d[..., 3] ** 2)).reshape(-1)
    ratio = ratio[torch.isfinite(ratio)]
    s = float(torch.quantile(ratio[:: max(1, ratio.numel() // 1000000)], case["magnify"])) if ratio.numel() else 1.0
    return (uv / s).float().contiguous(), (duv / s).float().contiguous()


def _xforms(case, seed):
    rng, n = _gen(seed, 4), case["layers"]
    s, t = rng.uniform(0.25, 4.0, n), rng.uniform(0, 2 * math.pi, n)
    return np.stack([s * np.cos(t), -s * np.sin(t), s * np.sin(t), s * np.cos(t)], -1).astype(np.float32)


def _texels(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 5)
    n, W = case["texels"] if case["op"] == "eval" else case["batch"], case["tex_w"]
    if n == W * W:      # the whole lattice, row by row, from a random corner
        i = torch.arange(n, device="cuda") + int(_gen(seed, 5).integers(0, W))
        return torch.stack([i % W, i // W], -1).int().contiguous()
    return torch.randint(0, W, (n, 2), generator=g, device="cuda", dtype=torch.int32)


_CTX = None


def _context():
    """One library context for the program's life."""
    global _CTX
    if _CTX is None:
        _CTX = ctf.Context(0)
    return _CTX


class _State:
    """What a program holds: the library objects and its own buffers."""

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        for t in getattr(self, "owned", ()):
            t.close()


def _texture(ctx, case, seed):
    """(texture, what has to be closed, in order)."""
    if case["tex"] == "sinusoids":
        t = ctx.sinusoid_texture(case["tex_w"], *_terms(case, seed))
    elif case["tex"] == "table":
        t = ctx.table_texture(_table(case, seed))
    else:
        d = ctx.decoder(case["l0"], case["l1"], HIDDEN, case["tex_w"], _params(case, seed))
        t = ctx.decoder_texture(d, PREC[case["precision"]])
        return t, [t, d]
    return t, [t]


def _method(case):
    return ctf.method(KIND[case["method"]], box=(case.get("box", 0),) * 2, k=case["k"],
                      fallback=FALLBACK[case.get("fallback", "stf1")], filter=FILTER[case["filter"]],
                      wave_shape=WAVE[case.get("wave", "8x8")])


def prepare(case, seed):
    ctx, op = _context(), case["op"]
    if op == "filter":
        tex, owned = _texture(ctx, case, seed)
        uv, duv = _scene(case, seed)
        return _State(case=case, ctx=ctx, tex=tex, owned=owned, uv=uv, duv=duv, meth=_method(case), seed=int(seed),
                      out=torch.empty((case["height"], case["width"], 4), device="cuda"))
    if op == "layers":
        owned, texs = [], []
        for l in range(case["layers"]):
            t, o = _texture(ctx, dict(case, tex="decoder"), seed + 1000 * (l + 1))
            texs.append(t)
            owned += o
        uv, duv = _scene(case, seed)
        return _State(case=case, ctx=ctx, texs=texs, owned=owned, uv=uv, duv=duv, meth=_method(case), seed=int(seed),
                      xf=_xforms(case, seed),
                      out=torch.empty((case["layers"], case["height"], case["width"], 4), device="cuda"))
    if op == "eval":
        tex, owned = _texture(ctx, case, seed)
        xy = _texels(case, seed)
        return _State(case=case, tex=tex, owned=owned, xy=xy, out=torch.empty((xy.shape[0], 4), device="cuda"))
    dec = ctx.decoder(case["l0"], case["l1"], HIDDEN, case["tex_w"], _params(case, seed))
    if op == "train":
        tex = ctx.sinusoid_texture(case["tex_w"], *_terms(case, seed))
        return _State(case=case, dec=dec, tex=tex, owned=[tex, dec], seed=int(seed),
                      trace=torch.empty(case["steps"], device="cuda"))
    xy = _texels(case, seed)
    target = _lattice_sinusoids(case, seed, xy).float().contiguous()
    return _State(case=case, dec=dec, owned=[dec], xy=xy, target=target)


def run(state):
    c = state.case
    if c["op"] == "filter":
        return state.ctx.filter(state.uv, state.duv, state.tex, state.meth, seed=state.seed, out=state.out)
    if c["op"] == "layers":
        return state.ctx.filter_layers(state.uv, state.duv, state.texs, state.xf, state.meth, seed=state.seed,
                                       out=state.out)
    if c["op"] == "eval":
        return state.tex.eval(state.xy, out=state.out)
    if c["op"] == "loss_grad":
        loss, grad = state.dec.loss_grad(state.xy, state.target, precision=PREC[c["precision"]])
        return {"loss": loss, "grad": grad}
    state.dec.train(state.tex, c["steps"], batch=c["batch"], lr=1e-3, seed=state.seed, precision=PREC[c["precision"]],
                    loss_trace=state.trace)
    return {"loss": state.trace, "params": state.dec.params()}


def work(case):
    """Bytes and operations of one pass: each input read and each output
    written once; the texel evaluations that the method cannot avoid (about
    one per minifying pixel and 0.4 (2x2 taps) or 0.76 (4x4) per magnifying
    one with one texel shared by the pixels of an 8x8 tile)."""
    op = case["op"]
    texel = MLP_FLOP
    if case.get("tex") == "sinusoids":
        texel = 4 * case["terms"] * TERM_FLOP
    elif case.get("tex") == "table":
        texel = 0
    latents = (case["l0"] ** 2 + case["l1"] ** 2) * CHANNELS * 2
    static = {"sinusoids": 64 * case.get("terms", 0), "table": 16 * case["tex_w"] ** 2}.get(case.get("tex"), latents)
    if op in ("filter", "layers"):
        n, px = case.get("layers", 1), case["width"] * case["height"]
        taps = 4 if case["filter"] == "bilinear" else 16
        per = {"bilinear4": taps, "stf1": 1}.get(
            case["method"], (1 - case["magnify"]) + case["magnify"] * (0.58 if taps == 4 else 1.09))
        return {"bytes": px * (24 + 16 * n) + n * static, "flops": n * px * per * (texel + 2 * 4 * taps / 2)}
    if op == "eval":
        return {"bytes": case["texels"] * 24 + static, "flops": case["texels"] * texel}
    params = 4 * (latents // 2 + 16 * 64 + 64 + 64 * 64 + 64 + 4 * 64 + 4)
    if op == "loss_grad":   # parameters read, gradient written, samples read
        return {"bytes": 2 * params + case["batch"] * 24, "flops": 3 * case["batch"] * MLP_FLOP}
    sample = 4 * case["terms"] * TERM_FLOP
    return {"bytes": case["steps"] * 6 * params, "flops": case["steps"] * case["batch"] * (3 * MLP_FLOP + sample)}


# ---------------------------------------------------------------------------
# the same in float64
# ---------------------------------------------------------------------------

def _lattice_sinusoids(case, seed, xy):
    """Procedural texels at xy in float64."""
    pqj, amp = _terms(case, seed)
    W, out = case["tex_w"], torch.empty((xy.shape[0], 4), dtype=torch.float64, device="cuda")
    x, y = xy[:, 0].double(), xy[:, 1].double()
    for c in range(4):
        acc = torch.zeros_like(x)
        for (p, q, j), a in zip(pqj[c].tolist(), amp[c].tolist()):
            acc += a * torch.sin((2 * math.pi / W) * torch.remainder(p * x + q * y + j, W))
        out[:, c] = 0.5 + 0.5 * acc
    return out


def _rounded(p, prec):
    return p.to(torch.float16 if prec == "fp16" else torch.bfloat16).double()


def _split(case, p):
    """The parts of the flat parameters: latents in the 16-bit type, weights
    likewise, biases as they are."""
    l0, l1, H, prec = case["l0"], case["l1"], HIDDEN, case["precision"]
    sizes = [l0 * l0 * 8, l1 * l1 * 8, 16 * H, H, H * H, H, H * 4, 4]
    lat0, lat1, W1, b1, W2, b2, W3, b3 = torch.split(p, sizes)
    r = lambda t: _rounded(t, prec)  # noqa: E731
    return [r(lat0).view(l0, l0, 8), r(lat1).view(l1, l1, 8), r(W1).view(16, H), b1.double(), r(W2).view(H, H),
            b2.double(), r(W3).view(H, 4), b3.double()]


def _decode(case, parts, xy):
    """Decoded texels at xy in float64 (differentiable in the parts)."""
    lat0, lat1, W1, b1, W2, b2, W3, b3 = parts
    feats = []
    for lat in (lat0, lat1):
        L = lat.shape[0]
        g = (xy.double() + 0.5) * (L / case["tex_w"]) - 0.5
        c = torch.floor(g)
        f, c = g - c, c.long()
        v = 0
        for dy in (0, 1):
            for dx in (0, 1):
                wgt = (f[:, 0] if dx else 1 - f[:, 0]) * (f[:, 1] if dy else 1 - f[:, 1])
                v = v + wgt[:, None] * lat[(c[:, 1] + dy) % L, (c[:, 0] + dx) % L]
        feats.append(v)
    h = torch.relu(torch.cat(feats, 1) @ W1 + b1)
    return torch.relu(h @ W2 + b2) @ W3 + b3


def _lattice(case, seed):
    """The texture's whole lattice in float64, [W][W][4]."""
    W = case["tex_w"]
    if case.get("tex") == "table":
        return torch.from_numpy(_table(case, seed)).cuda().double()
    i = torch.arange(W * W, device="cuda")
    xy = torch.stack([i % W, i // W], -1)
    if case.get("tex") == "sinusoids":
        return _lattice_sinusoids(case, seed, xy).view(W, W, 4)
    parts = _split(case, torch.from_numpy(_params(case, seed)).cuda())
    return torch.cat([_decode(case, parts, b) for b in xy.split(1 << 19)]).view(W, W, 4)


M32 = 0xFFFFFFFF


def _mul32(a, b):
    """Low 32 bits of a * b (int64 tensors or numbers below 2^32)."""
    return ((a & 0xFFFF) * b + (((a >> 16) * (b & 0xFFFF) & 0xFFFF) << 16)) & M32


def _pcg(v):
    s = (_mul32(v, 747796405) + 2891336453) & M32
    w = _mul32((s >> ((s >> 28) + 4)) ^ s, 277803737)
    return (w >> 22) ^ w


def _taps(x, filt):
    """float32 tap weights at x, in the documented op order."""
    if filt == "bilinear":
        return [1.0 - x, x]
    x2 = x * x
    x3, om = x2 * x, 1.0 - x
    if filt == "bspline":
        k = float(np.float32(1.0 / 6.0))
        return [((om * om) * om) * k, ((3.0 * x3 - 6.0 * x2) + 4.0) * k, (((-3.0 * x3 + 3.0 * x2) + 3.0 * x) + 1.0) * k,
                x3 * k]
    return [((2.0 * x2 - x3) - x) * 0.5, ((3.0 * x3 - 5.0 * x2) + 2.0) * 0.5, ((-3.0 * x3 + 4.0 * x2) + x) * 0.5,
            (x3 - x2) * 0.5]


def _cubic_draw(w, u):
    a = [t.abs() for t in w]
    p2 = a[0] + a[1]
    p3 = p2 + a[2]
    thr = u * (p3 + a[3])
    return (thr >= a[0]).long() + (thr >= p2).long() + (thr >= p3).long()


def _tiles(t, th, fill):
    """[H][W] -> [tiles][64 or 32], padded with ``fill``."""
    h, w = t.shape
    H, W = -(-h // th) * th, -(-w // 8) * 8
    p = torch.full((H, W), fill, dtype=t.dtype, device=t.device)
    p[:h, :w] = t
    return p.view(H // th, th, W // 8, 8).permute(0, 2, 1, 3).reshape(-1, th * 8)


def _pixels(ok, h, w, th):
    """Per-tile flags -> [H][W]."""
    ty, tx = -(-h // th), -(-w // 8)
    return ok.view(ty, 1, tx, 1).expand(ty, th, tx, 8).reshape(ty * th, tx * 8)[:h, :w]


def _successful(case, inA, x0, y0, F, O):
    """Per pixel: whether its wave's collaborative step succeeds."""
    th = 4 if case.get("wave") == "8x4" else 8
    A = _tiles(inA, th, False)
    big = 1 << 40
    ox, oy = _tiles(x0, th, 0) - O, _tiles(y0, th, 0) - O
    nA = A.sum(1)
    xmin, ymin = torch.where(A, ox, big).amin(1), torch.where(A, oy, big).amin(1)
    bw = torch.where(A, ox, -big).amax(1) + F - xmin
    bh = torch.where(A, oy, -big).amax(1) + F - ymin
    if case["method"] == "box":
        n, ok = bw * bh, (nA > 0)
        if case["box"]:
            ok &= (bw <= case["box"]) & (bh <= case["box"])
    else:
        n = torch.empty_like(nA)
        for b in range(0, A.shape[0], 16384):
            s = slice(b, b + 16384)
            keys = [torch.where(A[s], (oy[s] - ymin[s, None] + j) * (1 << 28) + (ox[s] - xmin[s, None] + i), -1)
                    for j in range(F) for i in range(F)]
            k = torch.sort(torch.cat(keys, 1), 1)[0]
            n[s] = (k[:, 1:] != k[:, :-1]).sum(1) + (k[:, 0] >= 0)
        ok = nA > 0
        if case["method"] == "mask":
            ok &= (bw <= 16) & (bh <= 16)
    return _pixels(ok & (n <= case["k"] * nA), *inA.shape, th)


def _filter64(case, uv, duv, lattice, seed, layer):
    """One filtered frame in float64 from the lattice."""
    W, filt = case["tex_w"], case["filter"]
    F, O = (2, 0) if filt == "bilinear" else (4, 1)
    h, w = uv.shape[:2]
    fx = (uv.double() * W - 0.5).float()
    active = torch.isfinite(uv).all(-1) & (fx.abs() < 16777216.0).all(-1)
    fx = torch.where(active[..., None], fx, torch.zeros_like(fx))
    fl = torch.floor(fx)
    st, c0 = fx - fl, fl.long()
    x0, y0 = c0[..., 0], c0[..., 1]
    d = duv * float(W)
    sq = lambda a, b: (a.double() * a.double() + (b * b).double()).float()  # noqa: E731
    magnify = (sq(d[..., 0], d[..., 1]) <= 1.0) & (sq(d[..., 2], d[..., 3]) <= 1.0)
    inA = active & magnify
    if case["method"] == "bilinear4":
        exact_px = active
    elif case["method"] == "stf1":
        exact_px = torch.zeros_like(active)
    else:
        exact_px = inA & _successful(case, inA, x0, y0, F, O)
    py, px = torch.meshgrid(torch.arange(h, device="cuda"), torch.arange(w, device="cuda"), indexing="ij")
    hh = _pcg(py ^ int(_pcg(torch.tensor(layer ^ ((seed >> 32) & M32)))))
    hh = _pcg((seed & M32) ^ _pcg(px ^ hh))
    u = [(v >> 8).float() * 2.0 ** -24 for v in (hh, _pcg(hh))]
    tx, ty = _taps(st[..., 0], filt), _taps(st[..., 1], filt)
    if F == 2:
        pick = (x0 + (u[0] < st[..., 0]), y0 + (u[1] < st[..., 1]))
    else:
        pick = (x0 - 1 + _cubic_draw(tx, u[0]), y0 - 1 + _cubic_draw(ty, u[1]))
    draw_px = active & ~exact_px
    out = lattice[pick[1] % W, pick[0] % W] * draw_px[..., None]
    wx = [t.double() for t in (tx if F == 4 else (1 - st[..., 0].double(), st[..., 0]))]
    wy = [t.double() for t in (ty if F == 4 else (1 - st[..., 1].double(), st[..., 1]))]
    for j in range(F):
        for i in range(F):
            wgt = (wx[i] * wy[j] * exact_px)[..., None]
            out += wgt * lattice[(y0 - O + j) % W, (x0 - O + i) % W]
    return out


def exact(case, seed):
    op = case["op"]
    if op in ("filter", "layers"):
        # Eq. 1 over a fallback wave's evaluated texels depends on its plan
        if case.get("fallback", "stf1") != "stf1" and case["method"] in ("list", "box", "mask"):
            return None
        uv, duv = _scene(case, seed)
        if op == "filter":
            return _filter64(case, uv, duv, _lattice(case, seed), int(seed), 0)
        out = torch.empty((case["layers"], case["height"], case["width"], 4), dtype=torch.float64, device="cuda")
        for l, m in enumerate(_xforms(case, seed).tolist()):
            # u' = fma(m01, v, m00 u): the inner product rounds to float32
            fma = lambda a, x, b, y: (b * y.double() + (a * x).double()).float()  # noqa: E731
            luv = torch.stack([fma(m[2 * r], uv[..., 0], m[2 * r + 1], uv[..., 1]) for r in (0, 1)], -1)
            lduv = torch.stack([fma(m[2 * r], duv[..., 2 * a], m[2 * r + 1], duv[..., 2 * a + 1])
                                for a in (0, 1) for r in (0, 1)], -1)
            out[l] = _filter64(case, luv, lduv, _lattice(case, seed + 1000 * (l + 1)), int(seed), l)
        return out
    if op == "eval":
        xy = _texels(case, seed).long() % case["tex_w"]
        if case["tex"] == "sinusoids":
            return _lattice_sinusoids(case, seed, xy)
        parts = _split(case, torch.from_numpy(_params(case, seed)).cuda())
        return torch.cat([_decode(case, parts, b) for b in xy.split(1 << 19)])
    if op == "train":
        return None     # the path of many optimiser steps has no exact value
    xy = _texels(case, seed).long()
    target = _lattice_sinusoids(case, seed, xy).float().double()
    parts = [p.requires_grad_() for p in _split(case, torch.from_numpy(_params(case, seed)).cuda())]
    loss = ((_decode(case, parts, xy) - target) ** 2).mean()
    loss.backward()
    return {"loss": loss.detach().view(1), "grad": torch.cat([p.grad.reshape(-1) for p in parts])}
