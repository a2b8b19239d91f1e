"""Every instance of the forward engines: a call that runs on it by name (asked of the library, so that a rule that takes the call
elsewhere is seen), against the oracle on sampled elements with the edges of tiles among them, at the gates of the other tests."""
import numpy as np
import pytest

import _util as U
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn
from paper_1909_09577_amd.inputs import LayerCfg


def gemm(nt, stride, kt, len_=False, stats=False, any_=False, pad_pair=False):
    return "conv_gemm_kernel<%d, %d, %d, %s, %s, %s, %s>" % (nt, stride, kt, *(str(v).lower() for v in (len_, stats, any_, pad_pair)))


def L(B, Cin, Cout, T, K, stride=1, dilation=1):
    pad = dilation * (K - 1) // 2
    return LayerCfg("layer", B, Cin, Cout, T, K, stride, dilation, pad, True, True, True, 61, T_out=orc.out_len(T, K, stride, dilation, pad))


# kernel without lengths, kernel with lengths, layer
UNROLLED = [(gemm(5, 1, c.K, any_=odd, len_=odd), gemm(5, 1, c.K, any_=odd, len_=True), c) for odd, c in [
    (False, L(2, 230, 77, 200, 11)), (False, L(2, 225, 187, 72, 13)), (False, L(8, 227, 541, 216, 17)), (False, L(6, 242, 204, 648, 21)),
    (False, L(10, 253, 843, 80, 25)), (False, L(8, 111, 771, 304, 29, dilation=2)),
    (True, L(2, 244, 88, 74, 11)), (True, L(7, 240, 34, 66, 13, dilation=2)), (True, L(16, 108, 143, 641, 17)), (True, L(37, 113, 148, 284, 21)),
    (True, L(9, 226, 935, 76, 25)), (True, L(34, 115, 84, 479, 29, dilation=2))]]
TAP_PAIRS = [(gemm(nt, c.stride, 0, any_=odd, pad_pair=pad), gemm(nt, c.stride, 0, any_=odd, pad_pair=pad), c) for nt, odd, pad, c in [
    (5, False, False, L(32, 256, 200, 808, 7)), (5, True, False, L(32, 256, 200, 801, 7)), (5, True, True, L(16, 480, 250, 801, 5)),
    (2, False, False, L(1, 104, 42, 16, 5)), (2, True, False, L(1, 134, 39, 20, 3, dilation=2)), (2, True, True, L(1, 134, 46, 16, 2)),
    (2, False, False, L(2, 66, 34, 208, 63, stride=2)), (2, True, False, L(2, 66, 54, 168, 64, stride=2)),
    (2, True, True, L(2, 65, 36, 180, 66, stride=2)), (2, True, True, L(4, 24, 100, 403, 1, stride=2))]]
POINTWISE = [("pointwise_gemm_kernel<false, 2, 5, 128>", "pointwise_gemm_kernel<true, 2, 5, 128>", L(2, 502, 302, 176, 1)),
             ("pointwise_gemm_kernel<true, 2, 5, 128>", "pointwise_gemm_kernel<true, 2, 5, 128>", L(2, 489, 313, 172, 1)),
             ("pointwise_gemm_kernel<false, 4, 4, 64>", "pointwise_gemm_kernel<true, 4, 4, 64>", L(26, 221, 1050, 168, 1)),
             ("pointwise_gemm_kernel<true, 4, 4, 64>", "pointwise_gemm_kernel<true, 4, 4, 64>", L(33, 270, 773, 172, 1))]
SPLIT = [(f"conv_split_kernel<{nt}, {c.stride}> {n}",) * 2 + (c,) for nt, n, c in [
    (2, "one", L(1, 64, 640, 264, 13)), (2, "parts", L(1, 512, 256, 203, 15)), (3, "one", L(29, 70, 522, 73, 3)), (3, "parts", L(1, 531, 648, 219, 1)),
    (4, "one", L(38, 40, 492, 104, 4, dilation=2)), (4, "parts", L(9, 520, 68, 206, 1)), (2, "one", L(3, 64, 256, 400, 11, stride=2)),
    (2, "parts", L(1, 596, 44, 91, 29, stride=2)), (3, "one", L(20, 40, 866, 144, 4, stride=2)), (3, "parts", L(22, 293, 37, 144, 29, stride=2))]]
CASES = UNROLLED + TAP_PAIRS + POINTWISE + SPLIT
STATS = [c for _, _, c in UNROLLED[:6]]


def short(name):
    if " in " not in name:
        return name
    return name.split(" in ")[0] + (" one" if name.endswith(" in 1 parts") else " parts")


def test_the_cases_reach_the_kernels_they_name():
    wrong = [(c.dims(), m, short(nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *c.dims(), flags=nm.NM_RELU, masked=m)), k)
             for plain, with_len, c in CASES for m, k in ((False, plain), (True, with_len))
             if short(nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *c.dims(), flags=nm.NM_RELU, masked=m)) != k]
    wrong += [(c.dims(), "statistics", nm.nm_conv1d_kernel_name(nm.NM_OP_BN_FWD, *c.dims(), flags=nm.NM_RELU)) for c in STATS
              if nm.nm_conv1d_kernel_name(nm.NM_OP_BN_FWD, *c.dims(), flags=nm.NM_RELU) != gemm(5, 1, c.K, stats=True)]
    assert not wrong, "\n".join(map(str, wrong))


def _sample(cfg, rng):
    """2048 elements, and all combinations of first, last and tile-edge channels and steps of the first and last item."""
    n = cfg.B * cfg.Cout * cfg.T_out
    ms = sorted({m for e in range(0, cfg.Cout + 64, 64) for m in (e - 1, e) if 0 <= m < cfg.Cout} | {cfg.Cout - 1})
    ts = sorted({t for w in (64, 96, 128, 160) for e in range(0, cfg.T_out + w, w) for t in (e - 1, e) if 0 <= t < cfg.T_out} | {cfg.T_out - 1})
    edges = [(b * cfg.Cout + m) * cfg.T_out + t for b in {0, cfg.B - 1} for m in ms[:8] + ms[-4:] for t in ts[:12] + ts[-8:]]
    return np.unique(np.concatenate([rng.integers(0, n, 2048), np.array(edges)]))


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[2].dims())))
def test_forward_kernels(case, masked):
    import torch
    cfg = case[2]
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    x, w = U.to_dev(inp, "x", "bf16"), U.to_dev(inp, "w", "bf16")
    scale, shift, res = (U.to_dev(inp, n, "bf16") for n in ("scale", "shift", "residual"))
    xh, lens = inp["x"].astype(np.float64), None
    if masked:  # poison behind the lengths; an item of one sample, one dead from the middle, the last one full
        n = np.array([max(1, cfg.T - 29 * b) for b in range(cfg.B)], dtype=np.int32)
        n[cfg.B // 2] = 1
        n[-1] = cfg.T if cfg.B > 1 else max(1, cfg.T - 5)
        lens = torch.from_numpy(n).cuda()
        for b in range(cfg.B):
            x[b, :, n[b]:] = float("nan")
            xh[b, :, n[b]:] = 0
    buf = torch.full((cfg.B * cfg.Cout * cfg.T_out + 128,), -7.0, dtype=torch.bfloat16, device="cuda")
    y = buf[64:-64].view(cfg.B, cfg.Cout, cfg.T_out)
    nm.nm_conv1d_block_fwd(x, w, scale, shift, res, y=y, relu=True, lengths=lens, **kw)
    got = U.to_host_f64(y).reshape(-1)
    idx = _sample(cfg, np.random.default_rng(9))
    ref = orc.block_fwd_at(xh, inp["w"].astype(np.float64), idx, inp["scale"], inp["shift"], inp["residual"], True, **kw)
    U.assert_close(got[idx], ref, "bf16", "y (sampled)")
    assert np.isfinite(got).all() and bool((buf[:64] == -7).all()) and bool((buf[-64:] == -7).all())


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", STATS, ids=lambda c: "x".join(map(str, c.dims())))
def test_statistics_of_ragged_tiles(cfg):
    """Mean and inverse deviation that the convolution's epilogue collects, against those of its stored output; z as above."""
    import torch
    inp = syn.make_inputs(cfg, "bf16")
    kw = U.geom_kw(cfg)
    x, w = U.to_dev(inp, "x", "bf16"), U.to_dev(inp, "w", "bf16")
    z, _, mean, invstd = nm.nm_conv1d_bn_fwd(x, w, U.to_dev(inp, "scale", "bf16"), U.to_dev(inp, "shift", "bf16"), relu=True, **kw)
    zf = z.double()
    assert torch.allclose(mean.double(), zf.mean(dim=(0, 2)), rtol=0, atol=1e-6)
    assert torch.allclose(invstd.double(), 1 / torch.sqrt(zf.var(dim=(0, 2), unbiased=False) + 1e-3), rtol=1e-5, atol=0)
    idx = _sample(cfg, np.random.default_rng(10))
    ref = orc.block_fwd_at(inp["x"].astype(np.float64), inp["w"].astype(np.float64), idx, None, None, None, False, **kw)
    U.assert_close(U.to_host_f64(z).reshape(-1)[idx], ref, "bf16", "z (sampled)")
