"""Float32 layers whose operands are split into three bfloat16 terms: at the edges of tiles, chunks and parts, at the gates of the other
float32 kernels (1e-5 of the result; no less exact than the plain kernels), and with operands of very different sizes."""
import numpy as np
import pytest

import _util as U
import test_gpu_f32 as base
from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm

pytestmark = pytest.mark.gpu

# around the edges of tiles of 32 channels x 32, 64 and 96 steps (test_f32_terms_instances.py says which tile and parts a size runs on, and
# reaches all of them); chunks of eight channels, the last one short; 64-step units of the weight gradient, its slices of 16 and its groups
# of 4, 8 and 12 taps
CASES = [base.L("cols_33", 1, 70, 40, 33, 11, pad=5, residual=True), base.L("cols_97", 9, 61, 230, 97, 13, pad=6),
         base.L("cols_193", 4, 200, 131, 193, 11, pad=5, residual=True), base.L("cols_127", 1, 130, 97, 127, 13, pad=6),
         base.L("cols_289", 5, 136, 257, 289, 11, pad=5), base.L("cols_311", 6, 97, 300, 311, 13, pad=6, residual=True),
         base.L("pad_wide", 2, 33, 34, 64, 11, pad=10), base.L("pad_none", 2, 40, 32, 80, 13, pad=0),
         base.L("taps_4", 2, 40, 48, 65, 4, pad=1), base.L("taps_8", 3, 31, 33, 129, 8, pad=3), base.L("taps_25", 2, 65, 32, 90, 25, pad=12)]


@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_edges(cfg, masked):
    base.test_float32_on_the_matrix_cores(cfg, masked)


@pytest.mark.parametrize("size", [2.0 ** -60, 2.0 ** 60, None], ids=["small", "large", "mixed"])
def test_sizes_of_operands(size):
    """Terms are exact at any size: the error stays that of float32 sums (1e-6 of the result where all channels have their own size,
    2e-7 being measured)."""
    import torch
    rng = np.random.default_rng(3)
    B, C, M, T, K = 2, 64, 48, 100, 11
    f = np.full(C, size) if size else 2.0 ** rng.integers(-50, 50, C)
    x = (rng.standard_normal((B, C, T)) * f[None, :, None]).astype(np.float32)
    w = (rng.standard_normal((M, C, K)) / f[None, :, None] / 26).astype(np.float32)
    dy = rng.standard_normal((B, M, T)).astype(np.float32)
    kw = dict(stride=1, dilation=1, pad=5)
    d = [torch.from_numpy(a).cuda() for a in (x, w, dy)]
    y = nm.nm_conv1d_block_fwd(d[0], d[1], None, None, None, relu=False, **kw)
    dx, _, dw = nm.nm_conv1d_bwd(d[0], d[2], d[1], relu=False, **kw)
    back = f[None, :, None]
    for got, ref, unit in ((y, orc.block_fwd(x, w, None, None, None, False, **kw), 1), (dx, orc.bwd_data(dy, w, T, **kw), back),
                           (dw, orc.bwd_weight(x, dy, K, **kw), 1 / back)):
        got, ref = U.to_host_f64(got) * unit, ref * unit
        assert np.linalg.norm(got - ref) <= 1e-6 * np.linalg.norm(ref)
