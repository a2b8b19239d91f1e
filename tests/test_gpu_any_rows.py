"""Rows that are no multiple of eight long on the matrix-core kernels: the pitched copies, the epilogue that writes such
rows in place and the mask pass that reads them, against the oracle at the gates of the other parity tests."""
import ctypes

import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg


def L(name, B, Cin, Cout, T, K, stride=1, dilation=1, pad=0, affine=True, relu=True, residual=False, seed=41):
    return LayerCfg(name, B, Cin, Cout, T, K, stride, dilation, pad, affine, relu, residual, seed,
                    T_out=orc.out_len(T, K, stride, dilation, pad))


CASES = [
    L("r_unrolled_1", 2, 128, 192, 321, 17, pad=8, residual=True),      # one element in the last group; unrolled kernel
    L("r_unrolled_7", 2, 256, 128, 167, 11, pad=5, residual=True),      # seven; a second time tile of seven steps
    L("r_private", 20, 128, 512, 1277, 11, pad=5, residual=True),       # private tiles (1280 of them)
    L("r_loop", 3, 72, 100, 333, 7, pad=3, residual=True),              # tap-pair loop, ragged channels
    L("r_narrow", 2, 64, 64, 50, 13, pad=6),                            # the 64-step tile
    L("r_short", 1, 32, 40, 3, 3, pad=1, residual=True),                # shorter than a group
    L("r_out_only", 2, 64, 64, 176, 4, pad=2, residual=True),           # T % 8 == 0, T_out = T + 1
    L("r_in_only", 2, 64, 64, 175, 4, pad=2, residual=True),            # T % 8 != 0, T_out = T + 1 = 176
    L("r_dil2", 2, 96, 80, 251, 29, dilation=2, pad=28),
    L("r_k1", 3, 136, 200, 331, 1, residual=True),
    L("r_k1_bigtile", 2, 136, 1000, 205, 1, residual=True),
    L("r_k1_bigtile_t", 2, 1000, 136, 205, 1, relu=False),
    L("r_k1_few", 2, 96, 29, 131, 1, affine=False, relu=False),
    L("r_stride2", 2, 64, 96, 403, 11, stride=2, pad=5),
    L("r_stride3", 2, 24, 40, 200, 5, stride=3, pad=2),
    L("r_shared_wgrad", 2, 1024, 512, 157, 17, pad=8, residual=True),   # the shared-staging weight-gradient kernel
]


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_rows_of_any_length(cfg, masked):
    import torch
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    lens = np.full(cfg.B, cfg.T, dtype=np.int32)
    x_bits = inp["x_bits"].copy()
    if masked:  # the last item full, the others ragged; poison behind them
        lens[:-1] = [max(0, cfg.T - 1 - 37 * b) for b in range(cfg.B - 1)]
        for b, n in enumerate(lens):
            x_bits[b, :, n:] = 0x7FC0
    ld = torch.from_numpy(lens).cuda() if masked else None
    x = torch.from_numpy(x_bits.view(np.int16)).cuda().view(torch.bfloat16)
    w, dy = U.to_dev(inp, "w", "bf16"), U.to_dev(inp, "dy", "bf16")
    scale = U.to_dev(inp, "scale", "bf16") if cfg.affine else None
    shift = U.to_dev(inp, "shift", "bf16") if cfg.affine else None
    res = U.to_dev(inp, "residual", "bf16") if cfg.residual else None
    hs = inp["scale"] if cfg.affine else None

    def guarded(shape, dtype=torch.bfloat16):  # an output between 64 sentinel values on either side
        n = int(np.prod(shape))
        buf = torch.full((n + 128,), -7.0, dtype=dtype, device="cuda")
        return buf, buf[64:64 + n].view(shape)

    def untouched(buf):
        return bool((buf[:64] == -7).all()) and bool((buf[-64:] == -7).all())

    act = (cfg.B, cfg.Cout, cfg.T_out)
    by, y = guarded(act)
    nm.nm_conv1d_block_fwd(x, w, scale, shift, res, y=y, relu=cfg.relu, lengths=ld, **kw)
    y_ref = orc.block_fwd_masked(inp["x"], inp["w"], lens, hs, inp["shift"] if cfg.affine else None,
                                 inp["residual"] if cfg.residual else None, cfg.relu, **kw)
    U.assert_close(U.to_host_f64(y), y_ref, "bf16", f"{cfg.name} y")
    assert untouched(by)

    y_saved = U.round_to_storage(y_ref, "bf16")
    ysv = U.arr_to_dev(y_saved, "bf16") if cfg.relu else None
    bx, dx = guarded((cfg.B, cfg.Cin, cfg.T))
    br, dres = guarded(act)
    nm.nm_conv1d_bwd_data(dy, w, cfg.T, y=ysv, scale=scale, dx=dx, dres=dres, relu=cfg.relu, lengths=ld, **kw)
    dw = nm.nm_conv1d_bwd_weight(x, dy, cfg.K, y=ysv, scale=scale, relu=cfg.relu, lengths=ld, **kw)
    dz, dres_ref = orc.epilogue_bwd(inp["dy"], y_saved.astype(np.float64) if cfg.relu else None, hs, cfg.relu)
    dx_ref = orc.bwd_data_masked(dz, inp["w"], cfg.T, lens, **kw)
    U.assert_close(U.to_host_f64(dx), dx_ref, "bf16", f"{cfg.name} dx")
    U.assert_close(U.to_host_f64(dw), orc.bwd_weight_masked(inp["x"], dz, cfg.K, lens, **kw), "bf16", f"{cfg.name} dw",
                   rms_bound=U.RMS_DW_BF16)
    np.testing.assert_array_equal(U.to_host_f64(dres), dres_ref)
    assert untouched(bx) and untouched(br)
    # one call for both gradients, and a workspace that only the plain kernels can do with
    dx1, dres1, dw1 = nm.nm_conv1d_bwd(x, dy, w, y=ysv, scale=scale, want_dres=True, relu=cfg.relu, lengths=ld, **kw)
    assert torch.equal(dx1, dx) and torch.equal(dres1, dres) and torch.equal(dw1, dw)
    if cfg.T * cfg.Cin * cfg.Cout * cfg.K < 1e8:
        small = torch.empty(2 * ((2 * dy.numel() + 255) // 256 * 256), dtype=torch.uint8, device="cuda")
        dx2, _, dw2 = nm.nm_conv1d_bwd(x, dy, w, y=ysv, scale=scale, relu=cfg.relu, lengths=ld, workspace=small, **kw)
        U.assert_close(U.to_host_f64(dx2), dx_ref, "bf16", f"{cfg.name} dx, small workspace")
        U.assert_close(U.to_host_f64(dw2), U.to_host_f64(dw), "bf16", f"{cfg.name} dw, small workspace", rms_bound=U.RMS_DW_BF16)
    if not masked and cfg.stride == 1:  # accumulation into dx: one rounding of old + gradient
        old = torch.randn(cfg.B, cfg.Cin, cfg.T, device="cuda").bfloat16()
        acc = old.clone()
        nm.nm_conv1d_bwd_data(dy, w, cfg.T, y=ysv, scale=scale, dx=acc, relu=cfg.relu, accumulate_dx=True, **kw)
        U.assert_close(U.to_host_f64(acc), U.to_host_f64(old) + dx_ref, "bf16", f"{cfg.name} dx accumulated")


FAKE = [ctypes.c_void_p(0x100000000000 + (i << 36)) for i in range(6)]


def test_a_workspace_of_the_plain_kernels_still_serves_rows_of_any_length():
    """No workspace was ever needed for the forward pass of such rows: a call without one is not refused (it ends at
    the launch, which has no device here), and neither is the entry point with the fixed scratch array."""
    big = (4, 512, 512, 8001, 17, 1, 1, 8)
    assert nm.nm_conv1d_workspace_bytes(nm.NM_OP_FWD, *big) > nm.NM_STATIC_SCRATCH_BYTES
    import torch
    if torch.cuda.is_available():
        pytest.skip("addresses without memory: not on a device")
    L_ = nm.lib()
    assert L_.nm_conv1d_block_fwd(*big, FAKE[0], FAKE[1], None, None, None, FAKE[2], 0, 0, None, 0, None) == nm.NM_ERR_DEVICE
    assert L_.nm_conv1d_block_fwd_static(*big, FAKE[0], FAKE[1], None, None, None, FAKE[2], 0, 0, None) == nm.NM_ERR_DEVICE
    # rows of 16-byte groups: as before
    even = big[:3] + (800,) + big[4:]
    assert L_.nm_conv1d_block_fwd(*even, FAKE[0], FAKE[1], None, None, None, FAKE[2], 0, 0, None, 0, None) == nm.NM_ERR_WORKSPACE
