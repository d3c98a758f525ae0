"""Batches of the decoder kernels that a tile does not fit, shown to occur.

A wave plans tiles behind each other on 256 rows and flushes first where a tile
like the last one would not fit.  Small and large tiles in random order defeat
that estimate: a tile of more than 256 - r rows drawn behind r rows of small
tiles is planned, found not to fit and planned again on an empty batch.  Each
of 3072 waves draws about eight tiles; where a tenth of the neighbouring draws
are such a pair, half of the waves meet one.  The tiles' rows come from the
oracle.  Checked as the other decoder tests: draws
and totals exact, colours within 1e-6.
"""
import numpy as np
import pytest

import ctf_synth as cs
import oracle as O

pytestmark = pytest.mark.gpu

TEX_W, SW, SH = 256, 1264, 1256      # 158 x 157 tiles, eight for each of 3072 waves


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


def frame(seed, large):
    """Head-on quads, half of them at magnification 1.5 and half at ``large``; a
    few pixels of every tile minify."""
    rng = np.random.default_rng(seed)
    ty, tx = SH // 8, SW // 8
    m = np.where(rng.uniform(size=(ty, 1, tx, 1)) < 0.5, 1.5, large)
    an = rng.uniform(0, np.pi / 2, m.shape)
    off = rng.uniform(0, TEX_W, (2,) + m.shape)
    yy, xx = np.arange(8).reshape(1, 8, 1, 1) + 0.5, np.arange(8).reshape(1, 1, 1, 8) + 0.5
    c, s = np.cos(an) / m, np.sin(an) / m
    uv = np.stack([((c * xx - s * yy) + off[0]) / TEX_W, ((s * xx + c * yy) + off[1]) / TEX_W], -1)
    duv = np.zeros((SH, SW, 4), np.float32)
    duv[rng.uniform(size=(SH, SW)) < 0.03, 0] = 1.0
    return uv.reshape(SH, SW, 2).astype(np.float32), duv


@pytest.mark.parametrize("kind,filt,large", [
    (2, 0, 0.3),     # List: four texels a pixel, boxes of 27 (sorted)
    (2, 1, 0.65),    # B-spline List: boxes of 16 and past it
    (4, 2, 0.72),    # Catmull-Rom Mask, some past the window (failing)
    (3, 0, 0.7),     # Box
])
def test_tiles_planned_again(G, kind, filt, large):
    ctf, ctx, torch = G
    uv, duv = frame(10 * kind + filt, large)
    dec = ctx.decoder(64, 16, 64, TEX_W, cs.decoder_init(64, 16, 64, seed=5, latent_range=0.5))
    tex = ctx.decoder_texture(dec, ctf.FP16)
    y, x = np.mgrid[0:TEX_W, 0:TEX_W]
    xy = np.stack([x.ravel(), y.ravel()], -1).astype(np.int32)
    table = tex.eval(torch.from_numpy(xy).cuda()).cpu().numpy().reshape(TEX_W, TEX_W, 4)
    okind = {2: O.LIST, 3: O.BOX, 4: O.MASK}[kind]
    o = O.filter_parallel(uv, duv, O.table_texture(table), O.method(okind, k=4, filter=filt), seed=9)
    st = o["stats"]
    rows, ok = st["evals"].astype(np.int64), (st["flags"] & O.TILE_OK) != 0
    # neighbours in a run: a small tile, then one that fits neither behind it
    # nor (were it like the small one) ahead of the estimate
    a, b = rows[:-1], rows[1:]
    again = (2 * a <= 256) & (a + b > 256)
    past = ok & ((st["bbw"] > 16) | (st["bbh"] > 16))
    print(f"rows {rows.min()}..{rows.max()}, again {again.mean():.2f}, successful past 16x16 {past.sum()}, "
          f"failing {(~ok).sum()}", flush=True)
    assert again.mean() > 0.1
    assert kind != 2 or past.sum() > 1000
    assert kind != 4 or ((~ok).sum() > 1000 and ok.sum() > 1000)
    gpu = [torch.from_numpy(t).cuda() for t in (uv, duv)]
    m = ctf.method(kind, k=4, filter=filt)
    fs, sx = ctf.frame_stats_buffer(), ctf.stf_buffer(SW, SH)
    out = ctx.filter(*gpu, tex, m, seed=9, frame_stats=fs, stf=sx)
    assert np.array_equal(sx.cpu().numpy(), o["stf"])
    err = np.abs(out.cpu().numpy().astype(np.float64) - o["out"]).max()
    assert err <= 1e-6, err
    fr = ctf.frame_stats_dict(fs)
    assert fr["evals"] == int(rows.sum()) and fr["tiles_ok"] == int(ok.sum())
    tex.close()
    dec.close()
