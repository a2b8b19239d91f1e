"""Stride-2 input gradient: both parities of the samples in one contraction, rows of any length, every alignment of the
two filters (pad and K even or odd), against the oracle at the gates of the other parity tests."""
import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg

CASES = [(3, 64, 256, T, K, pad) for T, K, pad in [
    (123, 11, 5), (122, 11, 4), (121, 10, 5), (160, 12, 0), (336, 11, 5), (9, 2, 1), (65, 3, 0), (64, 5, 7), (331, 7, 12)]]
CASES += [(2, 40, 72, 97, 11, 5), (20, 64, 256, 1002, 11, 5)]
# the engine for few tiles on the parities' contraction, in one part and in several, rows of any length (sums of 700 terms or
# more: of 95, weights rounded to bfloat16 put the largest of 2.5 million elements past the gate, 1.01e-2)
IN_SPLIT = {(27, 33, 129, 1229, 11, 5): "conv_split_kernel<3, 1> in 1 parts", (6, 33, 890, 199, 11, 5): "conv_split_kernel<4, 1> in 16 parts",
            (2, 24, 652, 163, 11, 5): "conv_split_kernel<2, 1> in "}
CASES += list(IN_SPLIT)


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_stride2_gradients(case, masked):
    import torch
    B, Cin, Cout, T, K, pad = case
    if case in IN_SPLIT:
        name = nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_DATA, B, Cin, Cout, T, K, 2, 1, pad, flags=nm.NM_RELU, masked=masked)
        assert name.startswith(IN_SPLIT[case]), name
    cfg = LayerCfg("stride2", B, Cin, Cout, T, K, 2, 1, pad, True, True, True, 47, T_out=orc.out_len(T, K, 2, 1, pad))
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    lens = np.full(B, T, dtype=np.int32)
    if masked:
        lens[:2] = [T - 1, (T + 1) // 2]
    ld = torch.from_numpy(lens).cuda() if masked else None
    x, w, dy = (U.to_dev(inp, n, "bf16") for n in ("x", "w", "dy"))
    scale = U.to_dev(inp, "scale", "bf16")
    ysv = U.to_dev(inp, "y_saved", "bf16")
    y_saved = U.to_host_f64(ysv)
    buf = torch.full((B * Cin * T + 128,), -7.0, dtype=torch.bfloat16, device="cuda")
    dx = buf[64:64 + B * Cin * T].view(B, Cin, T)
    dx1, dres1 = nm.nm_conv1d_bwd_data(dy, w, T, y=ysv, scale=scale, dx=dx, want_dres=True, relu=True, lengths=ld, **kw)
    dz, dres_ref = orc.epilogue_bwd(inp["dy"], y_saved, inp["scale"], True)
    dx_ref = orc.bwd_data_masked(dz, inp["w"], T, lens, **kw)
    U.assert_close(U.to_host_f64(dx), dx_ref, "bf16", "dx")
    np.testing.assert_array_equal(U.to_host_f64(dres1), dres_ref)
    assert bool((buf[:64] == -7).all()) and bool((buf[-64:] == -7).all())
    # one call for both gradients (one masked gradient feeds both), and the least workspace: the plain kernels
    dw = nm.nm_conv1d_bwd_weight(x, dy, K, y=ysv, scale=scale, relu=True, lengths=ld, **kw)
    dx2, dres2, dw2 = nm.nm_conv1d_bwd(x, dy, w, y=ysv, scale=scale, want_dres=True, relu=True, lengths=ld, **kw)
    assert torch.equal(dx2, dx) and torch.equal(dres2, dres1) and torch.equal(dw2, dw)
    U.assert_close(U.to_host_f64(dw), orc.bwd_weight_masked(inp["x"], dz, K, lens, **kw), "bf16", "dw", rms_bound=U.RMS_DW_BF16)
    if B * T < 2000:
        small = torch.empty((2 * dy.numel() + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
        dx3, _ = nm.nm_conv1d_bwd_data(dy, w, T, y=ysv, scale=scale, relu=True, lengths=ld, workspace=small, **kw)
        U.assert_close(U.to_host_f64(dx3), dx_ref, "bf16", "dx, small workspace")
