"""Calls next to each other in the range that a call accepts cost alike.

Each test times two calls of the same frame in turn, in one process, and bounds
the ratio of their best times; the bound lies between what the work of the two
calls explains and what the slow form of the call took.
"""
import numpy as np
import pytest

import ctf_synth as cs

pytestmark = pytest.mark.gpu

SW, SH = 1920, 1080


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


@pytest.fixture(scope="module")
def frame(G):
    """A rotated plane whose magnification runs from 0.7 to 3 across the
    screen, so tiles that share their texels and tiles that draw both count."""
    ctf, ctx, torch = G
    y, x = np.mgrid[0:SH, 0:SW].astype(np.float64)
    step = 1.4 / (1.0 + 3.3 * x / SW) / 512
    c, s = np.cos(0.4), np.sin(0.4)
    uv = np.stack([c * x * step - s * y * step, s * x * step + c * y * step], -1).astype(np.float32)
    duv = np.stack([c * step, s * step, -s * step, c * step], -1).astype(np.float32)
    return torch.from_numpy(uv).cuda(), torch.from_numpy(duv).cuda()


def times(torch, *calls):
    """Best time (us) of each call, the calls timed in turn."""
    best = [float("inf")] * len(calls)
    for call in calls:
        for _ in range(3):
            call()
    for _ in range(6):
        for i, call in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                call()
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("kind,k", [(2, 4), (3, 1), (4, 1)])
def test_8x4_terms_past_the_lds(G, frame, kind, k):
    """62 terms are the most that a workgroup holds in LDS.  With 63 they come
    from memory: 1.6 % more terms, and six instructions a term in place of five,
    9 lane slots in place of 8 (1.2 times); broadcast vector loads took 2.0
    times."""
    ctf, ctx, torch = G
    uv, duv = frame
    out = torch.empty((SH, SW, 4), device="cuda")
    m = ctf.method(kind, k=k, wave_shape=ctf.WAVE_8X4)
    texs = [ctx.sinusoid_texture(512, *cs.sinusoid_params(512, K, 64, seed=K)) for K in (62, 63)]
    near, past = times(torch, *[lambda t=t: ctx.filter(uv, duv, t, m, seed=3, out=out) for t in texs])
    print(f"62 terms {near:.1f} us, 63 terms {past:.1f} us")
    assert past <= 1.5 * near
    for t in texs:
        t.close()


@pytest.mark.parametrize("filt", [1, 2])
def test_frame_totals_of_a_cubic_frame(G, frame, filt):
    """Frame totals cost a line of atomics per wave, 8192 waves at most on this
    kernel, which the memory serves one after the other at about 15 ns: 0.12 ms
    on top of the frame.  One atomic per total took 1.1 ms."""
    ctf, ctx, torch = G
    uv, duv = frame
    out = torch.empty((SH, SW, 4), device="cuda")
    totals = ctf.frame_stats_buffer()
    tex = ctx.sinusoid_texture(512, *cs.sinusoid_params(512, 32, 64, seed=1))
    m = ctf.method(ctf.LIST, k=4, filter=filt)
    plain, counted = times(torch, lambda: ctx.filter(uv, duv, tex, m, seed=3, out=out),
                           lambda: ctx.filter(uv, duv, tex, m, seed=3, out=out, frame_stats=totals))
    print(f"plain {plain:.1f} us, with totals {counted:.1f} us")
    assert counted <= plain + 300
    tex.close()
