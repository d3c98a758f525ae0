"""Sums of the training kernels: the latent sums are left at zero by the kernel
that reads them, and the partial sums of the MLP gradient are reduced inside
the gradient and Adam kernels.

A batch's gradient is the mean of the gradients of its parts, and a part's
forward pass gives the same bits.  Where batch and parts are powers of two the
loss scale 2/(4n) changes by a power of two, so the back-propagated bf16 values
are the same too and only the float32 sums differ in order: at most 65536 / 16
terms in a row at 2^-24 each, 16 wide in norm: 1e-4 with room.  For other
sizes the rounding of the scaled residual and of two layers' signals differ,
u/2 each: 4 u.  One lost or doubled partial row changes the sum of n random
residuals by sqrt(1/rows) >= 0.06 of its norm.
"""
import numpy as np
import pytest

import ctf_synth as cs

pytestmark = pytest.mark.gpu

FP16, BF16 = 0, 1
U = {FP16: 2.0 ** -11, BF16: 2.0 ** -8}


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_2506_17770_amd as ctf
    ctx = ctf.Context(0)
    yield ctf, ctx, torch
    ctx.close()


def samples(torch, n, tex_w, seed):
    rng = np.random.default_rng(seed)
    xy = rng.integers(0, tex_w, (n, 2)).astype(np.int32)
    target = rng.uniform(0, 1, (n, 4)).astype(np.float32)
    return xy, target, torch.from_numpy(xy).cuda(), torch.from_numpy(target).cuda()


# tile edges, one workgroup and two, rows short of and past the unrolled
# eight, every wave of the largest launch
@pytest.mark.parametrize("hidden", [4, 12, 64])
@pytest.mark.parametrize("n,part", [(64, 16), (2048, 256), (65536, 4096), (17, 16), (65, 16), (4099, 256),
                                    (70001, 4096)])
def test_gradient_is_the_mean_of_its_parts(G, n, part, hidden):
    ctf, ctx, torch = G
    tex_w, l0, l1 = 64, 16, 4
    dec = ctx.decoder(l0, l1, hidden, tex_w, cs.decoder_init(l0, l1, hidden, seed=3, latent_range=0.5))
    _, _, xy, tg = samples(torch, n, tex_w, n)
    loss, grad = dec.loss_grad(xy, tg, precision=BF16)
    lsum, gsum = 0.0, np.zeros(dec.count)
    for i in range(0, n, part):
        m = min(part, n - i)
        l, g = dec.loss_grad(xy[i:i + m].contiguous(), tg[i:i + m].contiguous(), precision=BF16)
        lsum += float(l.cpu()[0]) * m / n
        gsum += g.cpu().numpy().astype(np.float64) * (m / n)
    # the loss comes from the forward pass alone
    assert abs(float(loss.cpu()[0]) - lsum) <= 1e-5 * lsum
    tol = 1e-4 if n & (n - 1) == 0 else 4 * U[BF16]
    grad = grad.cpu().numpy().astype(np.float64)
    for name, (o, m) in cs.decoder_layout(l0, l1, hidden).items():
        err, ref = np.linalg.norm(grad[o:o + m] - gsum[o:o + m]), np.linalg.norm(gsum[o:o + m])
        assert err <= tol * ref, (name, err / ref)
    dec.close()


@pytest.mark.parametrize("prec", [FP16, BF16])
def test_calls_leave_no_sums_behind(G, prec):
    """Gradient and training calls in any order, other batches and the other
    precision between them: each call's bits are those of a fresh decoder."""
    ctf, ctx, torch = G
    tex_w, l0, l1, H = 64, 16, 4, 32
    p = cs.decoder_init(l0, l1, H, seed=8, latent_range=0.5)
    pqj, amp = cs.sinusoid_params(tex_w, 8, 8, seed=2)
    tex = ctx.sinusoid_texture(tex_w, pqj, amp)
    _, _, xy, tg = samples(torch, 3001, tex_w, 1)
    _, _, xy2, tg2 = samples(torch, 129, tex_w, 2)
    whole = ctx.decoder(l0, l1, H, tex_w, p)
    first = whole.loss_grad(xy, tg, precision=prec)
    whole.train(tex, 6, batch=777, lr=1e-2, seed=4, precision=prec)
    last = whole.loss_grad(xy, tg, precision=prec)
    dec = ctx.decoder(l0, l1, H, tex_w, p)
    dec.loss_grad(xy2, tg2, precision=1 - prec)
    for a, b in zip(dec.loss_grad(xy, tg, precision=prec), first):
        assert torch.equal(a, b)
    dec.train(tex, 2, batch=777, lr=1e-2, seed=4, precision=prec)
    dec.loss_grad(xy2, tg2, precision=prec)
    dec.train(tex, 4, batch=777, lr=1e-2, seed=4, precision=prec)
    assert np.array_equal(dec.params(), whole.params())
    loss, grad = torch.empty(1, device="cuda"), torch.empty(dec.count, device="cuda")
    dec.loss_grad_noalloc(xy, tg, loss, grad, precision=prec)
    assert torch.equal(loss, last[0]) and torch.equal(grad, last[1])
    for o in (dec, whole, tex):
        o.close()
