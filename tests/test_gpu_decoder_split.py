"""The decoder's kernel where wavefronts share the channels of the same frames: shares of unequal length,
both sides of the lines between one, two and four, rows of any length, and the block forward on the same kernel."""
import numpy as np
import pytest

import _util as U
from oracle import decoder_oracle as dorc
from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn

CASES = [(1, 16, 29, 40, 1), (3, 256, 29, 96, 1), (1, 528, 32, 33, 4), (3, 1024, 29, 77, 4), (2, 272, 5, 9, 2), (8, 528, 29, 832, 4), (8, 528, 29, 840, 2),
         (16, 272, 29, 896, 2), (16, 272, 29, 904, 1), (16, 272, 29, 889, 2), (34, 608, 16, 456, 1), (1, 512, 7, 64, 2)]


def _bf16(a):
    return syn.bf16_bits_to_f32(syn.f32_to_bf16_bits(a.astype(np.float32)))


def test_the_lines():
    for B, Cin, Ncls, T, split in CASES:
        if T % 8 == 0:
            assert nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, B, Cin, Ncls, T, 1) == f"decoder_mfma_kernel<true, false, {split}>"


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_shared_channels(case):
    """Float32 sums of exact products: 5e-5 as in the other decoder tests; the block's output is bfloat16."""
    B, Cin, Ncls, T, _ = case
    gen = np.random.default_rng(2)
    x, w = _bf16(gen.standard_normal((B, Cin, T))), _bf16(gen.standard_normal((Ncls, Cin)) / np.sqrt(Cin))
    bias = gen.standard_normal(Ncls).astype(np.float32)
    xd, wd, bd = U.arr_to_dev(x, "bf16"), U.arr_to_dev(w, "bf16"), U.arr_to_dev(bias, "f32")
    got = nm.nm_decoder_logsoftmax_fwd(xd, wd, bd).cpu().numpy().astype(np.float64)
    mx, _ = U.err_metrics(got, dorc.decoder_logsoftmax(x, w, bias))
    assert mx <= 5e-5, mx
    if T % 8 == 0:
        y = nm.nm_conv1d_block_fwd(xd, wd.reshape(Ncls, Cin, 1), None, bd, relu=True)
        z = np.maximum(np.matmul(w.astype(np.float64), x) + bias[:, None], 0)
        U.assert_close(U.to_host_f64(y), z, "bf16", "y")
