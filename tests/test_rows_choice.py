"""Lines between conv_rows_kernel and the engine for few tiles, on either side of each, and the few-tap layers that run on the strided gradient's
instance."""
import pytest

import test_gpu_any_rows as rows
import test_gpu_rows_kernel as strided
from paper_1909_09577_amd import binding as nm


# row groups that are half full or less, with nearly empty last rounds and others; full groups
@pytest.mark.parametrize("dims,there", [((28, 638, 384, 528), False), ((26, 432, 320, 1272), False), ((24, 118, 300, 1352), False),
                                        ((20, 17, 300, 912), False), ((28, 43, 320, 1324), True), ((18, 470, 320, 1251), True),
                                        ((19, 432, 400, 953), True), ((33, 64, 256, 1000), True), ((32, 64, 256, 1600), True)], ids=str)
def test_strided_layers(dims, there):
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *dims, 11, 2, 1, 5, flags=nm.NM_RELU).startswith("conv_rows_kernel") == there


SIX = [((40, 50, 126, 128), False), ((46, 59, 104, 152), False), ((25, 36, 103, 968), True), ((18, 216, 101, 963), True), ((10, 300, 128, 960), True),
       ((9, 300, 128, 960), False), ((40, 64, 129, 1000), False), ((40, 64, 95, 1000), False)]


@pytest.mark.parametrize("dims,there", SIX, ids=str)
def test_six_taps(dims, there):
    B, R, M, T = dims
    name = nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *dims, 6, 1, 1, 3, flags=nm.NM_RELU)
    assert name.startswith("conv_rows_kernel<1, 2, 6>") == there
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_DATA, B, M, R, T, 6, 1, 1, 3, flags=nm.NM_RELU).startswith("conv_rows_kernel<1, 2, 6>") == there


# one, two and more chunks of channels, the last one short; rows of 16-byte groups and others; padding on either side and none.  (With lengths
# an item is 37 steps shorter than the one before it and the gate, 1e-2 of the result's rms plus its own size, takes the rms over the zeros
# behind them too: where all but 12 of 70 items are empty, that rms is 0.41 of the sums' own, and the six-sigma tail of the folded weights'
# rounding, 1e-2 of it, is 2e-2 there.  So no item is empty here.)
CASES = [rows.L("six", 25, 36, 103, 968, 6, pad=3, residual=True), rows.L("six_odd", 18, 216, 101, 963, 6, pad=2),
         rows.L("six_one_chunk", 23, 30, 128, 1189, 6, pad=0, residual=True), rows.L("six_gradient", 18, 97, 70, 1059, 6, pad=5)]


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_six_taps_results(cfg, masked):
    rows.test_rows_of_any_length(cfg, masked)


# row groups of two, one and three tiles that stay on the kernel, the last chunk short
PARTIAL = [strided.L(45, 70, 330, 386, False), strided.L(45, 40, 270, 389), strided.L(90, 33, 180, 257)]


@pytest.mark.parametrize("cfg", PARTIAL, ids=lambda c: "x".join(map(str, c.dims())))
def test_half_empty_row_groups(cfg):
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *cfg.dims(), flags=nm.NM_RELU).startswith("conv_rows_kernel<2, 4, 11>")


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", PARTIAL, ids=lambda c: "x".join(map(str, c.dims())))
def test_half_empty_row_groups_results(cfg, masked):
    strided.test_passes(cfg, masked)
