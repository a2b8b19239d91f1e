"""Calls of few tiles on the weights as they lie in memory: every filter length, tile width and direction of that kernel, at
edges of tiles, windows and tensors, against the oracle; and which calls take it."""
import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg

FWD, DGRAD = nm.NM_OP_FWD, nm.NM_OP_BWD_DATA


def L(B, Cin, Cout, T, K, dilation=1, pad=None, residual=True):
    pad = dilation * (K - 1) // 2 if pad is None else pad
    return LayerCfg("unpacked", B, Cin, Cout, T, K, 1, dilation, pad, True, True, residual, 17,
                    T_out=orc.out_len(T, K, 1, dilation, pad))


# tile width that the forward pass, the input gradient take (0: another engine)
CASES = [
    (L(1, 256, 256, 96, 11), 2, 2), (L(2, 128, 136, 77, 11, pad=0), 2, 0), (L(1, 128, 128, 9, 11), 2, 2), (L(3, 256, 256, 65, 11), 3, 3),
    (L(3, 256, 160, 65, 13), 2, 2), (L(1, 144, 192, 193, 13, dilation=2), 2, 2), (L(9, 256, 384, 66, 13), 3, 0), (L(2, 384, 384, 80, 13), 2, 3),
    (L(1, 256, 384, 129, 17, residual=False), 2, 0), (L(2, 192, 128, 161, 17, pad=3), 2, 2), (L(4, 512, 512, 72, 17), 3, 3),
    (L(2, 256, 200, 97, 21), 2, 0), (L(1, 512, 640, 333, 21), 2, 2), (L(3, 512, 640, 65, 21), 3, 3), (L(10, 640, 640, 132, 21), 2, 5),
    (L(1, 256, 256, 289, 25), 2, 0), (L(1, 768, 768, 601, 25), 2, 5), (L(3, 640, 768, 65, 25, residual=False), 3, 3), (L(7, 768, 768, 131, 25), 5, 0),
    (L(1, 256, 136, 100, 29), 2, 0), (L(2, 256, 128, 143, 29, dilation=2), 2, 0), (L(3, 768, 896, 67, 29, dilation=2), 3, 0),
    (L(7, 768, 896, 131, 29, dilation=2), 5, 0),
]


def width(op, c, **kw):
    name = nm.nm_conv1d_kernel_name(op, *c.dims(), flags=nm.NM_RELU, **kw)
    return int(name.split("conv_unpacked_kernel<")[1].split(",")[0]) if "conv_unpacked_kernel<" in name else 0


def test_the_cases_reach_the_kernel():
    got = [(c.dims(), width(FWD, c), width(DGRAD, c)) for c, _, _ in CASES]
    assert got == [(c.dims(), f, d) for c, f, d in CASES]
    assert {(c.K, f) for c, f, _ in CASES} >= {(k, 2) for k in (11, 13, 17, 21, 25, 29)}


def test_calls_it_does_not_take():
    """Channels of no whole chunk or tile, other filters, strides, many tiles, no room for the parts."""
    for c in (L(1, 250, 256, 96, 11), L(1, 112, 256, 96, 11), L(1, 256, 48, 96, 11), L(1, 256, 256, 96, 9), L(32, 256, 256, 800, 11)):
        assert width(FWD, c) == 0, c.dims()
    c = CASES[0][0]
    packed = (4 * 8 * 12 * 256 + 512) * 16
    assert width(FWD, c, workspace_bytes=packed) == 0
    assert 0 < nm.nm_conv1d_workspace_bytes(FWD, *c.dims()) - packed <= nm.NM_STATIC_SCRATCH_BYTES


def test_calls_that_are_faster_on_packed_weights():
    """The engine for few tiles in one part has no second launch: 20 us there, 31 here; two parts here: 34 there, 47 here."""
    for c in (L(10, 128, 1024, 203, 11), L(6, 128, 512, 935, 13), L(23, 256, 512, 203, 13), L(7, 192, 1024, 369, 13)):
        assert width(FWD, c) == 0, c.dims()
    assert width(FWD, L(23, 320, 768, 132, 13)) == 2  # (against the large engine two parts gain: 52 here, 72 there)


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", [c for c, _, _ in CASES], ids=lambda c: "x".join(map(str, c.dims())))
def test_forward_and_input_gradient(cfg, masked):
    """Within the gates of the other engines: products of bf16 are exact, sums are float32, results rounded once."""
    import torch
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    lens = np.full(cfg.B, cfg.T, dtype=np.int32)
    x_bits = inp["x_bits"].copy()
    if masked:  # poison behind the first item's length
        lens[0] = max(1, cfg.T - 45)
        x_bits[0, :, lens[0]:] = 0x7FC0
    ld = torch.from_numpy(lens).cuda() if masked else None
    n = x_bits.size  # x at an end of its allocation's poison: groups that run over the tensor's end
    buf = torch.full((n + 16,), float("nan"), dtype=torch.bfloat16, device="cuda")
    x = buf[8:8 + n].view(cfg.B, cfg.Cin, cfg.T)
    x.copy_(torch.from_numpy(x_bits.view(np.int16)).cuda().view(torch.bfloat16))
    w, dy = U.to_dev(inp, "w", "bf16"), U.to_dev(inp, "dy", "bf16")
    scale, shift = U.to_dev(inp, "scale", "bf16"), U.to_dev(inp, "shift", "bf16")
    res = U.to_dev(inp, "residual", "bf16") if cfg.residual else None
    guard = torch.full((nm.nm_conv1d_workspace_bytes(FWD, *cfg.dims(), nm.NM_BF16, nm.NM_RELU) + 256,), 255, dtype=torch.uint8, device="cuda")
    y = nm.nm_conv1d_block_fwd(x, w, scale, shift, res, relu=True, lengths=ld, workspace=guard[:-256], **kw)
    assert bool((guard[-256:] == 255).all())
    y_ref = orc.block_fwd_masked(inp["x"], inp["w"], lens, inp["scale"], inp["shift"], inp["residual"] if cfg.residual else None, True, **kw)
    U.assert_close(U.to_host_f64(y), y_ref, "bf16", "y")
    if not masked and cfg.Cin * cfg.Cout * cfg.K < 10e6:
        ys = torch.full_like(y, float("nan"))
        nm.nm_conv1d_block_fwd_static(x, w, scale, shift, res, y=ys, relu=True, **kw)
        assert torch.equal(ys, y)
    y_saved = U.round_to_storage(y_ref, "bf16")
    ysv = U.arr_to_dev(y_saved, "bf16")
    dx = nm.nm_conv1d_bwd_data(dy, w, cfg.T, y=ysv, scale=scale, relu=True, lengths=ld, **kw)[0]
    dz, _ = orc.epilogue_bwd(inp["dy"], y_saved.astype(np.float64), inp["scale"], True)
    dx_ref = orc.bwd_data_masked(dz, inp["w"], cfg.T, lens, **kw)
    U.assert_close(U.to_host_f64(dx), dx_ref, "bf16", "dx")
    dx1, dres, _ = nm.nm_conv1d_bwd(x, dy, w, y=ysv, scale=scale, relu=True, want_dres=True, lengths=ld, **kw)
    assert torch.equal(dx1, dx)
    if not masked:  # a sum in place, and no mask pass at all
        old = torch.randn(cfg.B, cfg.Cin, cfg.T, device="cuda").bfloat16()
        acc = old.clone()
        nm.nm_conv1d_bwd_data(dres, w, cfg.T, scale=scale, dx=acc, accumulate_dx=True, **kw)
        U.assert_close(U.to_host_f64(acc), U.to_host_f64(old) + dx_ref, "bf16", "dx accumulated")


@pytest.mark.gpu
def test_replayed_in_a_graph():
    import torch
    cfg = CASES[0][0]
    inp = syn.make_inputs(cfg, "bf16")
    x, w, scale, shift = (U.to_dev(inp, n, "bf16") for n in ("x", "w", "scale", "shift"))
    y, ws = torch.empty(cfg.B, cfg.Cout, cfg.T_out, dtype=torch.bfloat16, device="cuda"), torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    call = lambda: nm.nm_conv1d_block_fwd(x, w, scale, shift, y=y, relu=True, workspace=ws, **U.geom_kw(cfg))
    want = call().clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        y.zero_()
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
