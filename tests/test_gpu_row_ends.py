"""The last group of rows that are no multiple of eight long, read with the row's last eight elements and written in pieces of four, two and
one: every remainder, rows shorter than a group and rows of one group and a bit, with and without lengths."""
import pytest

import test_gpu_any_rows as base

pytestmark = pytest.mark.gpu

CASES = [base.L(f"end_{T}", 3, 64, 72, T, 11, pad=5, residual=True) for T in (1, 5, 7, 9, 10, 11, 12, 13, 14, 15, 63, 65)]
CASES += [base.L("end_k1", 2, 70, 129, 97, 1, residual=True), base.L("end_split", 1, 256, 256, 203, 11, pad=5, residual=True),
          # at most 32 output channels: a wavefront, two and four that share the channels of the same steps
          base.L("end_few", 2, 96, 29, 9, 1, residual=True), base.L("end_few_2", 2, 272, 20, 203, 1, residual=True),
          base.L("end_few_4", 1, 1024, 29, 97, 1, relu=False)]


@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_row_ends(cfg, masked):
    base.test_rows_of_any_length(cfg, masked)
