"""Branches of the per-lane kernels (8x8 waves, and two 8x4 tiles per wave).

The full filter of a procedural texture evaluates the four bilinear taps, or a
row of cubic taps, together where the terms are staged in LDS as floats and
the texture is at most 2048 wide, and tap by tap elsewhere.  Both give the
values of the single-texel evaluation, so the frame equals, bit for bit, the
frame of the table that holds them.

Random quads, one magnification per tile, then put tiles with a set, with a
set past the 16x16 window (sorted) and with a failing wave side by side, so
that the two halves of a wave of 8x4 tiles go different ways; odd tile counts
leave a half without a tile.  Checked against the oracle with the bar of the
other filter tests (decisions exact, colours within 1e-6).
"""
import numpy as np
import pytest

import ctf_synth as cs
import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


def table_of(G, tex, W):
    ctf, ctx, torch = G
    y, x = torch.meshgrid(torch.arange(W, dtype=torch.int32, device="cuda"),
                          torch.arange(W, dtype=torch.int32, device="cuda"), indexing="ij")
    xy = torch.stack([x.reshape(-1), y.reshape(-1)], -1).contiguous()
    return ctx.table_texture(tex.eval(xy).cpu().numpy().reshape(W, W, 4))


@pytest.mark.parametrize("W,K", [(64, 1), (64, 62), (64, 63), (2048, 3), (2048, 32), (4096, 5)])
def test_full_filter_equals_the_table_bitwise(G, W, K):
    ctf, ctx, torch = G
    pqj, amp = cs.sinusoid_params(W, K, W // 4, seed=W + K)
    tex = ctx.sinusoid_texture(W, pqj, amp)
    tab = table_of(G, tex, W)
    rng = np.random.default_rng(K)
    sh, sw = 83, 117
    uv = rng.uniform(-2, 2, (sh, sw, 2))
    edge = rng.uniform(size=(sh, sw, 2)) < 0.5      # taps across the texture's edge
    uv[edge] = np.round(uv[edge]) + rng.uniform(-3, 3, int(edge.sum())) / W
    uv = torch.from_numpy(uv.astype(np.float32)).cuda()
    duv = torch.zeros(sh, sw, 4, device="cuda")
    for shape in (ctf.WAVE_8X8, ctf.WAVE_8X4):
        for filt in (ctf.FILTER_BILINEAR, ctf.FILTER_BSPLINE, ctf.FILTER_CATMULL_ROM):
            m = ctf.method(ctf.BILINEAR4, filter=filt, wave_shape=shape)
            a, b = ctx.filter(uv, duv, tex, m), ctx.filter(uv, duv, tab, m)
            assert torch.equal(a, b), (shape, filt, (a - b).abs().max().item())
    tab.close()
    tex.close()


def tile_quads(tw, th, tiles_x, tiles_y, W, seed):
    """Screen of tw x th quads at log-uniform magnification 0.3 .. 4."""
    rng = np.random.default_rng(seed)
    m = np.exp(rng.uniform(np.log(0.3), np.log(4.0), (tiles_y, 1, tiles_x, 1)))
    an = rng.uniform(0, np.pi / 2, m.shape)
    off = rng.uniform(0, W, (2,) + m.shape)
    yy, xx = np.arange(th).reshape(1, th, 1, 1) + 0.5, np.arange(tw).reshape(1, 1, 1, tw) + 0.5
    c, s = np.cos(an) / m, np.sin(an) / m
    uv = np.stack([((c * xx - s * yy) + off[0]) / W, ((s * xx + c * yy) + off[1]) / W], -1)
    uv = uv.reshape(tiles_y * th, tiles_x * tw, 2).astype(np.float32)
    duv = np.zeros(uv.shape[:2] + (4,), np.float32)
    duv[rng.uniform(size=duv.shape[:2]) < 0.05, 0] = 1.0     # some lanes minify
    return uv, duv


@pytest.mark.parametrize("th", [8, 4])
@pytest.mark.parametrize("kind,filt,k,fb", [(2, 0, 1, 0), (2, 0, 2, 1), (2, 1, 4, 2), (4, 0, 1, 2), (4, 2, 2, 1),
                                            (3, 0, 1, 2)])
def test_mixed_tiles(G, th, kind, filt, k, fb):
    from test_gpu_filter import compare, run_gpu
    from test_gpu_wave32 import run_w32
    ctf, ctx, torch = G
    W = 64
    for K in (5, 64):       # terms staged in LDS, read from memory
        pqj, amp = cs.sinusoid_params(W, K, 8, seed=K)
        tex = ctx.sinusoid_texture(W, pqj, amp)
        uv, duv = tile_quads(8, th, 31, 17, W, seed=10 * kind + filt)
        uv, duv = uv[:-1], duv[:-1]
        shape = ctf.WAVE_8X8 if th == 8 else ctf.WAVE_8X4
        m = ctf.method(kind, k=k, fallback=fb, filter=filt, wave_shape=shape)
        g = (run_gpu if th == 8 else run_w32)(G, uv, duv, tex, m, seed=21)
        okind = {2: O.LIST, 3: O.BOX, 4: O.MASK}[kind]
        o = O.filter(uv, duv, O.sinusoid_texture(W, pqj, amp), O.method(okind, k=k, fallback=fb, filter=filt),
                     seed=21, tile=(8, th), lists=True, stf=True)
        ok = (o["stats"]["flags"] & O.TILE_OK) != 0
        assert ok.sum() >= 20 and (~ok).sum() >= 20
        compare(g, o, f"8x{th} {kind} {filt} K={K}")
        # without the optional outputs (another instantiation): the same colours
        plain = ctx.filter(torch.from_numpy(uv).cuda(), torch.from_numpy(duv).cuda(), tex, m, seed=21)
        assert np.array_equal(plain.cpu().numpy(), g["out"])
        tex.close()
