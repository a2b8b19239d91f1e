"""Where a backward call makes both gradients in parts, their sums share the last launch, unless the input gradient's kernels are timed: the
timer's events enclose its sum.  On the device: the bits of the two separate calls, with few and with many parts and rows of any length."""
import pytest

import _launches as la
from paper_1909_09577_amd import binding as nm

CALLS = [{"call": "bwd", "dims": (1, 256, 256, 200, 11, 1, 1, 5), "flags": nm.NM_RELU}, {"call": "bwd", "dims": (2, 640, 768, 83, 1, 1, 1, 0), "flags": nm.NM_RELU}]


@pytest.mark.parametrize("call", CALLS, ids=lambda c: str(c["dims"]))
def test_launches(call):
    (status, seq), (st, timed) = la.run([call, dict(call, timer=nm.NM_OP_BWD_DATA)])
    assert status == st == nm.NM_OK
    kernels = [k for _, k, _ in seq]
    assert kernels[-1] == "both_sums_kernel" and "split_reduce_kernel" not in kernels and "wgrad_reduce4_kernel" not in kernels
    a, b = ([i for i, (kind, what, _) in enumerate(timed) if (kind, what) == ("event", e)] for e in (la.START, la.STOP))
    assert [k for _, k, _ in timed[a[0] + 1:b[0]]][-1] == "split_reduce_kernel" and timed[-1][1] == "wgrad_reduce4_kernel"


@pytest.mark.gpu
@pytest.mark.parametrize("B,Cin,Cout,T,K", [(1, 256, 256, 200, 11), (3, 256, 320, 77, 13), (2, 512, 640, 83, 1), (4, 768, 256, 100, 1), (1, 258, 256, 64, 1),
                                            (2, 640, 640, 95, 21)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_bits_of_the_separate_calls(B, Cin, Cout, T, K, accumulate):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    x, w, dy, y = r(B, Cin, T), r(Cout, Cin, K) * 0.02, r(B, Cout, T), r(B, Cout, T).clamp_min(0)
    scale = torch.rand(Cout, device="cuda", generator=g) + 0.5
    kw = dict(stride=1, dilation=1, pad=K // 2, relu=True)
    old_x, old_w = r(B, Cin, T), torch.randn(Cout, Cin, K, device="cuda", generator=g)
    dx, dw, dx2, dw2 = old_x.clone(), old_w.clone(), old_x.clone(), old_w.clone()
    nm.nm_conv1d_bwd(x, dy, w, y=y, scale=scale, dx=dx, dw=dw, accumulate=accumulate, accumulate_dx=accumulate, **kw)
    nm.nm_conv1d_bwd_data(dy, w, T, y=y, scale=scale, dx=dx2, accumulate_dx=accumulate, **kw)
    nm.nm_conv1d_bwd_weight(x, dy, K, y=y, scale=scale, dw=dw2, accumulate=accumulate, **kw)
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)
