"""Batch statistics and the passes around them on rows of any length: the last group of a row begins inside the one before it, so
its first elements must count once; rows shorter than a group go element by element; addresses that are no multiple of 16 bytes."""
import pytest

import _util as U
from paper_1909_09577_amd import binding as nm

pytestmark = pytest.mark.gpu


def _case(B, C, T, dtype, offset):
    import torch
    g = torch.Generator().manual_seed(B * 1000 + C + T)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32

    def make(*shape):
        flat = torch.zeros(offset + B * C * T, dtype=t)
        v = flat[offset:].view(B, C, T)
        v.copy_(torch.randn(B, C, T, generator=g))
        return flat.cuda()[offset:].view(B, C, T)
    w = torch.randn(C, C, 3, generator=g).mul_((3 * C) ** -0.5).to(t).cuda()
    f = [torch.rand(C, generator=g).add_(0.5).cuda(), torch.randn(C, generator=g).mul_(0.1).cuda()]
    return make(), w, f[0], f[1], make(), make()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,C,T,offset", [(2, 8, 3, 0), (3, 8, 4, 1), (3, 16, 7, 0), (2, 16, 8, 3), (9, 24, 9, 1), (5, 16, 15, 0),
                                          (17, 8, 129, 0), (1, 16, 2047, 1), (9, 16, 1030, 1), (3, 16, 8200, 0)])
def test_statistics_and_gradients(B, C, T, offset, dtype):
    import torch
    x, w, gamma, beta, res, dy = _case(B, C, T, dtype, offset)
    kw = dict(pad=1, relu=True)
    z, y, mean, invstd = nm.nm_conv1d_bn_fwd(x, w, gamma, beta, res, eps=1e-3, **kw)
    zd, n = z.double().cpu(), B * T
    mu, var = zd.mean((0, 2)), zd.var((0, 2), unbiased=False)
    is_ = (var + 1e-3) ** -0.5
    # mean, invstd: sums of at most 8 terms in float, the rest in double, of values up to about 4
    assert (mean.double().cpu() - mu).abs().max() <= 1e-6 and ((invstd.double().cpu() - is_) / is_).abs().max() <= 4e-6
    col = lambda v: v.double().cpu()[None, :, None]
    m, i = col(mean), col(invstd)
    want = ((zd - m) * i * col(gamma) + col(beta) + res.double().cpu()).clamp(min=0)
    step = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -21  # half a unit in the last place; float: a few roundings
    assert ((y.double().cpu() - want).abs() <= step * want.abs() + 4e-6).all()
    # gradients: dy as given; everything from the stored z, y and statistics
    dx, dres, dw, dgamma, dbeta = nm.nm_conv1d_bn_bwd(x, w, gamma, z, y, mean, invstd, dy, want_dres=True, **kw)
    g = torch.where(y.double().cpu() > 0, dy.double().cpu(), 0.0)
    zh = (zd - m) * i
    assert torch.equal(dres.double().cpu(), g)
    sb, sg = g.sum((0, 2)), (g * zh).sum((0, 2))
    bound = 1e-6 * (g.abs().sum((0, 2)) + (g * zh).abs().sum((0, 2))) + 1e-6
    assert ((dbeta.double().cpu() - sb).abs() <= bound).all() and ((dgamma.double().cpu() - sg).abs() <= bound).all()
    dz = col(gamma) * i * (g - (sb / n)[None, :, None] - zh * (sg / n)[None, :, None])
    xd = x.double().cpu().requires_grad_()
    wd = w.double().cpu().requires_grad_()
    torch.nn.functional.conv1d(xd, wd, padding=1).backward(dz)
    # dz is rounded to the storage type and contracted: 3*C products a sum, dx stored; dw in float
    dev = 2.0 ** -8 if dtype == "bf16" else 1e-5
    rel = lambda a, b: ((a.double().cpu() - b).pow(2).mean() / b.pow(2).mean().clamp(min=1e-12)).sqrt()
    assert rel(dx, xd.grad) <= dev and rel(dw, wd.grad) <= dev
