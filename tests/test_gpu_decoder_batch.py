"""Edges of the batched decoder kernels and of the 32-texel decode.

A wave of the batched kernels plans up to four tiles on at most 256 rows
before it decodes them, and a tile whose rows do not fit behind the others
(or that sorts its set, for the bicubic filters) is planned again on an empty
batch.  A screen with more tiles than the chip holds waves, each tile a
head-on quad at its own magnification, mixes tiles of a few rows with tiles
of up to 256 rows and boxes past the 16x16 window, so that batches end in
every way.  Checked against the oracle filtering the GPU-decoded lattice:
draws and frame counts exact, colours within 1e-6 (the float32 weighting bound
the other decoder tests use).
"""
import numpy as np
import pytest

import ctf_synth as cs
import oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-6
TEX_W = 256


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


def decoder_texture(G, prec, seed=5):
    ctf, ctx, torch = G
    dec = ctx.decoder(64, 16, 64, TEX_W, cs.decoder_init(64, 16, 64, seed=seed, latent_range=0.5))
    return dec, ctx.decoder_texture(dec, prec)


def lattice(G, tex):
    _, _, torch = G
    ys, xs = np.mgrid[0:TEX_W, 0:TEX_W]
    xy = np.ascontiguousarray(np.stack([xs.ravel(), ys.ravel()], -1).astype(np.int32))
    return torch.from_numpy(xy).cuda(), tex


def quads(sw, sh, seed, lo, hi):
    """uv of a screen whose 8x8 tiles are quads at log-uniform magnification
    lo..hi; one tile in eight has a share of minifying pixels."""
    rng = np.random.default_rng(seed)
    tx, ty = (sw + 7) // 8, (sh + 7) // 8
    m = np.exp(rng.uniform(np.log(lo), np.log(hi), (ty, 1, tx, 1)))
    an = rng.uniform(0, np.pi / 2, (ty, 1, tx, 1))
    off = rng.uniform(0, TEX_W, (2, ty, 1, tx, 1))
    yy, xx = np.arange(8).reshape(1, 8, 1, 1) + 0.5, np.arange(8).reshape(1, 1, 1, 8) + 0.5
    c, s = np.cos(an) / m, np.sin(an) / m
    u = ((c * xx - s * yy) + off[0]) / TEX_W
    v = ((s * xx + c * yy) + off[1]) / TEX_W
    uv = np.stack([u, v], -1).reshape(ty * 8, tx * 8, 2)[:sh, :sw].astype(np.float32)
    duv = np.zeros((ty, 8, tx, 8, 4), np.float32)
    mini = (rng.uniform(size=(ty, 1, tx, 1)) < 0.125) & (rng.uniform(size=(ty, 8, tx, 8)) < 0.5)
    duv[mini, 0] = 1.0
    return np.ascontiguousarray(uv), np.ascontiguousarray(duv.reshape(ty * 8, tx * 8, 4)[:sh, :sw])


@pytest.mark.parametrize("prec", [0, 1])
def test_eval_tails(G, prec):
    """Texel counts around the 16-row and 32-row tiles: every count gives the
    same bits as the whole lattice."""
    _, _, torch = G
    dec, tex = decoder_texture(G, prec)
    xy, _ = lattice(G, tex)
    whole = tex.eval(xy)
    for n in (1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 2047, 40001):
        assert torch.equal(tex.eval(xy[:n].contiguous()), whole[:n]), n
    tex.close()
    dec.close()


@pytest.mark.parametrize("kind,filt,k,lo,hi", [
    (2, 0, 4, 0.55, 12.0),    # List: up to 256 rows a tile
    (2, 0, 4, 0.3, 2.0),      # List: boxes past the window (sorted sets)
    (4, 0, 2, 0.8, 8.0),      # Mask with failing waves
    (3, 0, 4, 0.8, 12.0),     # Box
    (1, 0, 1, 0.5, 8.0),      # one tap per pixel
    (2, 1, 4, 0.7, 12.0),     # B-spline List, some sorted
    (4, 2, 4, 1.0, 12.0),     # Catmull-Rom Mask
])
def test_mixed_tiles(G, kind, filt, k, lo, hi):
    ctf, ctx, torch = G
    sw, sh = 1261, 797        # 158 x 100 tiles, ragged on both sides
    uv, duv = quads(sw, sh, 100 * kind + filt, lo, hi)
    dec, tex = decoder_texture(G, ctf.FP16)
    xy, _ = lattice(G, tex)
    table = tex.eval(xy).cpu().numpy().reshape(TEX_W, TEX_W, 4)
    gpu = [torch.from_numpy(t).cuda() for t in (uv, duv)]
    m = ctf.method(kind, k=k, filter=filt)
    fs, sx = ctf.frame_stats_buffer(), ctf.stf_buffer(sw, sh)
    out = ctx.filter(*gpu, tex, m, seed=9, frame_stats=fs, stf=sx)
    okind = {1: O.STF1, 2: O.LIST, 3: O.BOX, 4: O.MASK}[kind]
    o = O.filter_parallel(uv, duv, O.table_texture(table), O.method(okind, k=k, filter=filt), seed=9)
    st, fr = o["stats"], ctf.frame_stats_dict(fs)
    rows = st["evals"].astype(np.int64)
    print(f"rows a tile: {rows.min()}..{rows.max()}", flush=True)
    assert np.array_equal(sx.cpu().numpy(), o["stf"])
    err = np.abs(out.cpu().numpy().astype(np.float64) - o["out"]).max()
    assert err <= TOL, err
    assert fr["evals"] == int(rows.sum())
    assert fr["rows"] >= fr["evals"] and fr["rows"] % 16 == 0
    # the layered launch with one untransformed layer: the same bits
    lay = ctx.filter_layers(*gpu, [tex], np.eye(2, dtype=np.float32)[None], m, seed=9)
    assert torch.equal(lay[0], out)
    tex.close()
    dec.close()
