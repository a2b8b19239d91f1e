"""Weight gradient with shared staging: how many parts a call takes, and the units of a padded batch (items of no length among
them, more items than lanes of a wavefront) against the oracle."""
import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg


def L(B, Cin, Cout, T, K, dilation=1):
    pad = dilation * (K - 1) // 2
    return LayerCfg("wgrad", B, Cin, Cout, T, K, 1, dilation, pad, True, True, False, 5, T_out=orc.out_len(T, K, 1, dilation, pad))


# the parts of many layers' worth of tiles cost more than idle CUs do; few tiles still fill the chip with them
@pytest.mark.parametrize("dims,name", [
    ((16, 640, 640, 800, 21, 1, 1, 10), "wgrad_shared_kernel<21, 1, false> in 1 parts"),
    ((16, 640, 768, 296, 25, 1, 1, 12), "wgrad_shared_kernel<13, 1, false> in 1 parts"),
    ((3, 768, 768, 112, 25, 1, 1, 12), "wgrad_fast_kernel<5, 1> in 1 parts"),
    # few channels: the parts of whole rounds
    ((32, 1024, 16, 24, 25, 1, 1, 12), "wgrad_shared_kernel<13, 1, false> in 4 parts"),
    ((35, 512, 16, 28, 25, 1, 1, 12), "wgrad_shared_kernel<13, 1, false> in 8 parts"),
    ((32, 512, 512, 800, 17, 1, 1, 8), "wgrad_shared_kernel<17, 1, false> in 2 parts"),
    ((32, 256, 256, 800, 11, 1, 1, 5), "wgrad_shared_kernel<11, 1, false> in 8 parts"),
    ((1, 256, 256, 96, 11, 1, 1, 5), "wgrad_fast_kernel<6, 1> in 1 parts")], ids=str)
def test_parts(dims, name):
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *dims) == name


CASES = [(L(70, 256, 256, 24, 11), None), (L(70, 256, 320, 96, 11), None), (L(64, 256, 256, 41, 11), None), (L(3, 384, 512, 170, 17), [170, 0, 81]),
         (L(5, 320, 640, 88, 21), [88, 80, 79, 1, 88]), (L(3, 512, 512, 96, 29, dilation=2), [40, 96, 7]),
         (L(200, 256, 256, 40, 11), [0] * 130 + [33] * 70), (L(129, 256, 320, 88, 13), [88, 5, 0] * 43)]


def test_the_cases_run_on_the_kernel_with_shared_staging():
    for c, _ in CASES:
        assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *c.dims(), masked=True).startswith("wgrad_shared_kernel<"), c.dims()


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0].dims())))
def test_weight_gradient(case, masked):
    import torch
    cfg, given = case
    inp = syn.make_inputs(cfg, "bf16")
    lens = np.full(cfg.B, cfg.T, dtype=np.int32)
    if masked:
        lens = np.array(given if given else [(37 * b) % (cfg.T + 1) for b in range(cfg.B)], dtype=np.int32)
    x = U.to_dev(inp, "x", "bf16")
    for b in range(cfg.B):
        x[b, :, lens[b]:] = float("nan")
    dy, scale = U.to_dev(inp, "dy", "bf16"), U.to_dev(inp, "scale", "bf16")
    ld = torch.from_numpy(lens).cuda() if masked else None
    dw = nm.nm_conv1d_bwd_weight(x, dy, cfg.K, scale=scale, lengths=ld, **U.geom_kw(cfg))
    dz, _ = orc.epilogue_bwd(inp["dy"], None, inp["scale"], False)
    U.assert_close(U.to_host_f64(dw), orc.bwd_weight_masked(inp["x"], dz, cfg.K, lens, **U.geom_kw(cfg)), "bf16", "dw", rms_bound=U.RMS_DW_BF16)


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg,parts,now", [(L(4, 640, 640, 392, 21), 5, 1), (L(13, 384, 512, 288, 17), 8, 2), (L(12, 384, 384, 240, 13), 7, 3),
                                           (L(3, 768, 896, 400, 29, dilation=2), 3, 1)],
                         ids=lambda c: "x".join(map(str, c.dims())) if isinstance(c, LayerCfg) else "")
def test_fewer_parts_are_no_less_exact(cfg, parts, now, masked):
    """Fewer parts than whole rounds over the CUs would take: their sums are no longer chains than those.  A chain of n
    roundings of growing sums, each 2^-24 / sqrt(3) of its sum, ends sqrt(n / 2) of that off (measured: 0.8 of it); a chain over
    the whole part is the root of parts / now as far off, which the gate of the other tests does not see."""
    import torch
    d = cfg.dims()
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, dy = (torch.randn(cfg.B, c, cfg.T, device="cuda", generator=gen).bfloat16() for c in (cfg.Cin, cfg.Cout))
    lens = torch.full((cfg.B,), cfg.T, dtype=torch.int32, device="cuda")
    if masked:
        lens[1:] = cfg.T - 100
    keep = torch.arange(cfg.T, device="cuda") < lens[:, None]
    pad = torch.nn.functional.pad((x * keep[:, None, :]).double(), (cfg.pad, cfg.pad))
    g = dy.double().transpose(0, 1).reshape(cfg.Cout, -1)
    ref = torch.stack([g @ pad[:, :, k * cfg.dilation:k * cfg.dilation + cfg.T].transpose(1, 2).reshape(-1, cfg.Cin)
                       for k in range(cfg.K)], dim=2)
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *d, masked=masked).endswith(f" in {now} parts")
    dw = nm.nm_conv1d_bwd_weight(x, dy, cfg.K, lengths=lens if masked else None, **U.geom_kw(cfg))
    steps = 5 * cfg.B * -(-cfg.T // 80) // parts
    assert ((dw.double() - ref).norm() / ref.norm()).item() <= 2**-24 / 3**0.5 * (steps / 2) ** 0.5


@pytest.mark.gpu
def test_units_of_many_items_are_not_walked():
    """256 padded items take no longer than 256 whole ones but for what it costs to look the lengths up (1.1 times); a walk over
    the items for every unit took 20 times as long."""
    import torch
    B, C, T, K = 256, 256, 80, 11
    x, dy = torch.randn(B, C, T, device="cuda").bfloat16(), torch.randn(B, C, T, device="cuda").bfloat16()
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, B, C, C, T, K, 1, 1, 5, masked=True).startswith("wgrad_shared_kernel<11, 1, true>")
    ws = torch.empty(nm.nm_conv1d_workspace_bytes(nm.NM_OP_BWD_WEIGHT, B, C, C, T, K, 1, 1, 5), dtype=torch.uint8, device="cuda")
    dw = torch.empty(C, C, K, device="cuda")

    def best(lengths):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(6):
            ev[0].record()
            for _ in range(10):
                nm.nm_conv1d_bwd_weight(x, dy, K, dw=dw, pad=5, lengths=lengths, workspace=ws)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]))
        return min(times)

    whole, padded = best(None), best(torch.full((B,), T, dtype=torch.int32, device="cuda"))
    assert padded < 3 * whole, (padded, whole)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [L(1, 512, 512, 70, 17), L(5, 512, 640, 193, 21), L(1, 768, 768, 64, 25), L(4, 512, 512, 321, 17)],
                         ids=lambda c: "x".join(map(str, c.dims())))
def test_fp8_weight_gradient_in_any_number_of_parts(cfg):
    """One part up to several (the fewest where a part costs more than idle CUs), the gate of the other 8-bit weight gradients."""
    import test_gpu_fp8 as T8
    got, ref = T8.run_wgrad_case(cfg, accumulate=True)
    mx, rr = U.err_metrics(got, ref)
    assert mx <= T8.WGRAD_TOL and rr <= T8.WGRAD_RMS, (mx, rr)


# a workspace with room for fewer parts than are asked for now (what these calls asked for under other rules: weight gradient,
# both gradients): as many as there is room for
SMALLER = [(L(9, 192, 512, 613, 17), 34765824, 43990016, "wgrad_fast_kernel<6, 1> in 4 parts"),
           (L(8, 256, 320, 168, 13), 22528000, 28835840, "wgrad_shared_kernel<13, 1, false> in 4 parts"),
           (L(5, 256, 384, 1001, 13), 27021312, 33652736, "wgrad_fast_kernel<5, 1> in 4 parts"),
           (L(16, 320, 512, 312, 25), 21626880, 35266560, "wgrad_fast_kernel<5, 1> in 1 parts"),
           (L(4, 320, 128, 640, 25), 17039360, 19832832, "wgrad_shared_kernel<13, 1, false> in 4 parts")]


@pytest.mark.parametrize("cfg,ws_w,ws_both,name", SMALLER, ids=lambda c: "x".join(map(str, c.dims())) if isinstance(c, LayerCfg) else "")
def test_less_room_takes_fewer_parts(cfg, ws_w, ws_both, name):
    assert nm.nm_conv1d_workspace_bytes(nm.NM_OP_BWD_WEIGHT, *cfg.dims(), nm.NM_BF16, nm.NM_RELU) > ws_w
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *cfg.dims(), workspace_bytes=ws_w) == name


@pytest.mark.gpu
@pytest.mark.parametrize("both", [False, True], ids=["weight", "both"])
@pytest.mark.parametrize("cfg,ws_w,ws_both,name", SMALLER, ids=lambda c: "x".join(map(str, c.dims())) if isinstance(c, LayerCfg) else "")
def test_weight_gradient_in_less_room(cfg, ws_w, ws_both, name, both):
    import torch
    inp = syn.make_inputs(cfg, "bf16")
    x, dy, scale, w = (U.to_dev(inp, k, "bf16") for k in ("x", "dy", "scale", "w"))
    n = ws_both if both else ws_w
    buf = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    kw = dict(scale=scale, workspace=buf[:n], **U.geom_kw(cfg))
    dz, _ = orc.epilogue_bwd(inp["dy"], None, inp["scale"], False)
    if both:
        dx, _, dw = nm.nm_conv1d_bwd(x, dy, w, **kw)
        U.assert_close(U.to_host_f64(dx), orc.bwd_data(dz, inp["w"], cfg.T, **U.geom_kw(cfg)), "bf16", "dx")
    else:
        dw = nm.nm_conv1d_bwd_weight(x, dy, cfg.K, **kw)
    assert (buf[n:] == 0xA5).all()
    U.assert_close(U.to_host_f64(dw), orc.bwd_weight(inp["x"], dz, cfg.K, **U.geom_kw(cfg)), "bf16", "dw", rms_bound=U.RMS_DW_BF16)
