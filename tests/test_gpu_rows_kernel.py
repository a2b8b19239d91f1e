"""The strided first layer on workgroups whose wavefronts have rows and columns of their own: names on either side of the lines that send a
call there, and forward pass and both gradients at the edges of its tiles against the oracle."""
import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg


def L(B, Cin, Cout, T, res=True, stride=2, K=11, pad=5):
    return LayerCfg("rows", B, Cin, Cout, T, K, stride, 1, pad, True, True, res, 71, T_out=orc.out_len(T, K, stride, 1, pad))


@pytest.mark.parametrize("op,dims,there", [(nm.NM_OP_FWD, (32, 64, 256, 1600), True), (nm.NM_OP_FWD, (25, 64, 256, 1000), True),
                                           (nm.NM_OP_FWD, (24, 64, 256, 1000), False), (nm.NM_OP_FWD, (32, 64, 128, 1600), False),
                                           (nm.NM_OP_BWD_DATA, (20, 64, 256, 1000), True), (nm.NM_OP_BWD_DATA, (19, 64, 256, 1000), False),
                                           (nm.NM_OP_BWD_DATA, (32, 128, 256, 1600), False)], ids=str)
def test_line(op, dims, there):
    assert nm.nm_conv1d_kernel_name(op, *dims, 11, 2, 1, 5, flags=nm.NM_RELU).startswith("conv_rows_kernel") == there


# row groups that are not full, one and several chunks, the last one short, odd and even rows, one step in the last column
CASES = [L(29, 64, 256, 850), L(70, 40, 200, 389), L(41, 70, 330, 386, False), L(84, 33, 180, 257), L(27, 64, 256, 770, pad=4), L(70, 48, 72, 259)]


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "x".join(map(str, c.dims())))
def test_passes(cfg, masked):
    import torch
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    x, w, dy = (U.to_dev(inp, n, "bf16") for n in ("x", "w", "dy"))
    scale, shift = U.to_dev(inp, "scale", "bf16"), U.to_dev(inp, "shift", "bf16")
    res = U.to_dev(inp, "residual", "bf16") if cfg.residual else None
    xh, dyh, lens = inp["x"].astype(np.float64), inp["dy"].astype(np.float64), None
    n = np.full(cfg.B, cfg.T, dtype=np.int32)
    if masked:  # poison behind the lengths; an item of one sample, one dead from the middle
        n = np.maximum(1, cfg.T - 11 * np.arange(cfg.B, dtype=np.int32))
        n[cfg.B // 2] = 1
        lens = torch.from_numpy(n).cuda()
        for b in range(cfg.B):
            x[b, :, n[b]:] = float("nan")
            xh[b, :, n[b]:] = 0
    y = nm.nm_conv1d_block_fwd(x, w, scale, shift, res, relu=True, lengths=lens, **kw)
    rng = np.random.default_rng(4)

    def sample(rows, cols):
        edges = [(b * rows + m) * cols + t for b in (0, cfg.B // 2, cfg.B - 1) for m in {0, 63, 64, rows - 1} if m < rows
                 for t in {0, 1, 62, 63, 64, 127, 128, cols - 2, cols - 1} if t < cols]
        return np.unique(np.concatenate([rng.integers(0, cfg.B * rows * cols, 2048), np.array(edges)]))

    idx = sample(cfg.Cout, cfg.T_out)
    ref = orc.block_fwd_at(xh, inp["w"].astype(np.float64), idx, inp["scale"], inp["shift"], inp["residual"] if cfg.residual else None, True, **kw)
    U.assert_close(U.to_host_f64(y).reshape(-1)[idx], ref, "bf16", "y (sampled)")
    assert bool(torch.isfinite(y).all())
    dx, _ = nm.nm_conv1d_bwd_data(dy, w, cfg.T, scale=scale, relu=False, lengths=lens, **kw)
    idx = sample(cfg.Cin, cfg.T)
    ref = orc.bwd_data_at(dyh * inp["scale"].astype(np.float64)[None, :, None], inp["w"].astype(np.float64), cfg.T, idx, **kw)
    bi, t = idx // (cfg.Cin * cfg.T), idx % cfg.T
    got, there = U.to_host_f64(dx).reshape(-1)[idx], t < n[bi]
    # the gate scales by the result's rms: over the positions that have one (with lengths a sixth of them; counted among them the zeros
    # behind a length halve the rms and so twice the rounding of 2^-8 crosses 1e-2)
    U.assert_close(got[there], ref[there], "bf16", "dx (sampled)")
    assert (got[~there] == 0).all()
