"""Loss/gradient passes recorded into a graph: a replay gives the same bits
whatever ran or failed between the recording and the replay.

A pass fails here the way it does in a program: an earlier HIP call of the
thread left an error, which the library's first launch check reports, so the
forward and backward kernel has run and the one that reads and clears its sums
has not.  Gradients are bitwise reproducible, so every comparison is exact.
"""
import numpy as np
import pytest

import ctf_synth as cs

pytestmark = pytest.mark.gpu

TEX_W, L0, L1, H = 64, 16, 4, 32


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


def batch(torch, n, seed):
    rng = np.random.default_rng(seed)
    return (torch.from_numpy(rng.integers(0, TEX_W, (n, 2)).astype(np.int32)).cuda(),
            torch.from_numpy(rng.uniform(0, 1, (n, 4)).astype(np.float32)).cuda())


def decoder(ctx):
    return ctx.decoder(L0, L1, H, TEX_W, cs.decoder_init(L0, L1, H, seed=8, latent_range=0.5))


def record(G, dec, xy, tg, prec):
    """A graph of one pass and the buffers that it writes."""
    ctf, ctx, torch = G
    loss, grad = torch.zeros(1, device="cuda"), torch.zeros(dec.count, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dec.loss_grad_noalloc(xy, tg, loss, grad, precision=prec)
    return graph, loss, grad


def failing_pass(G, dec, xy, tg, prec):
    ctf, ctx, torch = G
    torch.cuda.synchronize()
    assert ctf.lib.hipSetDevice(1 << 20) != 0       # refused by the host; the error stays with the thread
    with pytest.raises(ctf.CtfError):
        dec.loss_grad(xy, tg, precision=prec)
    torch.cuda.synchronize()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [17, 4099])
def test_replay_after_a_failed_pass(G, n, prec):
    ctf, ctx, torch = G
    dec = decoder(ctx)
    xy, tg = batch(torch, n, n)
    xy2, tg2 = batch(torch, 129, 2)
    want = dec.loss_grad(xy, tg, precision=prec)
    want2 = dec.loss_grad(xy2, tg2, precision=prec)
    graph, loss, grad = record(G, dec, xy, tg, prec)
    for _ in range(2):
        failing_pass(G, dec, xy2, tg2, prec)
        for _ in range(2):                          # the replay next to the failure, and one after it
            loss.zero_(), grad.zero_()
            graph.replay()
            assert torch.equal(loss, want[0]) and torch.equal(grad, want[1])
        # an eager pass next to the failure, and one after it
        failing_pass(G, dec, xy, tg, prec)
        for _ in range(2):
            got = dec.loss_grad(xy2, tg2, precision=prec)
            assert torch.equal(got[0], want2[0]) and torch.equal(got[1], want2[1])
    dec.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_first_pass_recorded(G, prec):
    """A decoder whose first pass is a graph's, replayed with eager passes and
    training between the replays."""
    ctf, ctx, torch = G
    xy, tg = batch(torch, 1000, 1)
    other = decoder(ctx)
    want = other.loss_grad(xy, tg, precision=prec)
    dec = decoder(ctx)
    graph, loss, grad = record(G, dec, xy, tg, prec)
    for _ in range(3):
        loss.zero_(), grad.zero_()
        graph.replay()
        assert torch.equal(loss, want[0]) and torch.equal(grad, want[1])
        got = dec.loss_grad(xy, tg, precision=prec)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    for d in (dec, other):
        d.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_failed_change_of_precision(G, prec):
    """A call in the other precision that fails while it rewrites the 16-bit
    copies leaves no half-written copies behind."""
    ctf, ctx, torch = G
    dec = decoder(ctx)
    xy, tg = batch(torch, 300, 5)
    want = dec.loss_grad(xy, tg, precision=prec)
    failing_pass(G, dec, xy, tg, 1 - prec)
    got = dec.loss_grad(xy, tg, precision=prec)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    dec.close()
