"""What a call launches, seen without a GPU: a refused launch is reported whichever it is, and the timer's events enclose the
kernels that the header says they do."""
import pytest

import _launches as la
from paper_1909_09577_amd import binding as nm

R, F32 = nm.NM_RELU, nm.NM_F32
# one call of every kind of route
CALLS = {
    "split engine, parts": {"call": "fwd", "dims": (1, 768, 640, 203, 1, 1, 1, 0), "flags": R},
    "split engine, parts, static": {"call": "static", "dims": (1, 768, 640, 203, 1, 1, 1, 0), "flags": R},
    "split engine, stride 2": {"call": "fwd", "dims": (1, 596, 44, 91, 29, 2, 1, 14)},
    "split engine, gradient": {"call": "bwd_data", "dims": (1, 640, 768, 203, 1, 1, 1, 0), "flags": R},
    "unpacked": {"call": "fwd", "dims": (1, 256, 256, 200, 11, 1, 1, 5), "with": ["res"]},
    "unpacked gradient": {"call": "bwd_data", "dims": (1, 256, 256, 200, 11, 1, 1, 5), "flags": R, "with": ["dres"]},
    "large": {"call": "fwd", "dims": (32, 256, 256, 800, 11, 1, 1, 5), "masked": True},
    "odd rows": {"call": "fwd", "dims": (16, 384, 384, 777, 13, 1, 1, 6)},
    "both gradients": {"call": "bwd", "dims": (32, 256, 256, 800, 11, 1, 1, 5), "flags": R, "with": ["dres"]},
    "both gradients, odd rows": {"call": "bwd", "dims": (16, 384, 384, 777, 13, 1, 1, 6), "flags": R, "masked": True},
    "both gradients, few tiles": {"call": "bwd", "dims": (1, 256, 256, 200, 11, 1, 1, 5), "flags": R},
    "both gradients, stride 2": {"call": "bwd", "dims": (32, 64, 256, 1600, 11, 2, 1, 5), "flags": R},
    "both gradients, K=1": {"call": "bwd", "dims": (32, 896, 1024, 800, 1, 1, 1, 0), "flags": R},
    "both gradients, two calls": {"call": "bwd", "dims": (4, 64, 96, 160, 5, 1, 3, 6), "flags": R},
    "weight gradient": {"call": "bwd_weight", "dims": (4, 384, 384, 160, 13, 1, 1, 6), "flags": R},
    "BatchNorm": {"call": "bn_fwd", "dims": (16, 640, 640, 800, 21, 1, 1, 10), "flags": R},
    "BatchNorm, few tiles": {"call": "bn_fwd", "dims": (1, 256, 256, 200, 11, 1, 1, 5), "flags": R},
    "BatchNorm gradients": {"call": "bn_bwd", "dims": (4, 256, 256, 200, 11, 1, 1, 5), "flags": R},
    "float32": {"call": "fwd", "dims": (4, 256, 256, 400, 11, 1, 1, 5), "dtype": F32, "flags": R},
    "float32, shared": {"call": "fwd", "dims": (1, 256, 256, 60, 11, 1, 1, 5), "dtype": F32, "flags": R},
    "float32, shared, gradients": {"call": "bwd", "dims": (1, 256, 256, 60, 11, 1, 1, 5), "dtype": F32, "flags": R},
    "8 bits": {"call": "fp8_fwd", "dims": (4, 512, 512, 200, 17, 1, 1, 8), "flags": R},
    "8 bits, gradients": {"call": "fp8_bwd", "dims": (4, 512, 512, 200, 17, 1, 1, 8), "flags": R, "with": ["dres"]},
    "decoder": {"call": "decoder", "dims": (2, 1024, 29, 77)},
    "plain": {"call": "bwd", "dims": (2, 8, 8, 40, 3, 3, 1, 1), "flags": R},
}


@pytest.fixture(scope="module")
def whole():
    return dict(zip(CALLS, la.run(list(CALLS.values()))))


@pytest.mark.parametrize("name", CALLS)
def test_a_refused_launch_is_reported(name, whole):
    status, seq = whole[name]
    assert status == nm.NM_OK and seq and all(kind == "launch" for kind, _, _ in seq)
    got = la.run([dict(CALLS[name], refuse=i + 1) for i in range(len(seq))])
    for (st, s), (_, kernel, _) in zip(got, seq):
        assert any(kind == "refused" and k == kernel for kind, k, _ in s)
        assert st == nm.NM_ERR_DEVICE, f"{kernel} refused, status {st}"


def test_the_timer_counts_the_sum_of_the_parts():
    """A convolution's pair of events encloses the pass that adds up and finishes its parts, and nothing else."""
    pairs = [(name, op, kernels) for name, op, kernels in [
        ("split engine, parts", nm.NM_OP_FWD, ["conv_split_kernel", "split_reduce_kernel"]),
        ("unpacked", nm.NM_OP_FWD, ["conv_unpacked_kernel", "split_reduce_kernel"]),
        ("unpacked gradient", nm.NM_OP_BWD_DATA, ["conv_unpacked_kernel", "split_reduce_kernel"]),
        ("float32", nm.NM_OP_FWD, ["f32_conv_kernel"]),
        ("float32, shared", nm.NM_OP_FWD, ["f32_conv_kernel", "f32_split_finish_kernel"]),
        ("float32, shared, gradients", nm.NM_OP_BWD_DATA, ["f32_conv_kernel", "f32_split_finish_kernel"]),
        ("float32, shared, gradients", nm.NM_OP_BWD_WEIGHT, ["f32_wgrad_kernel"])]]
    for (name, op, kernels), (status, seq) in zip(pairs, la.run([dict(CALLS[n], timer=op) for n, op, _ in pairs])):
        assert status == nm.NM_OK
        a, b = ([i for i, (kind, what, _) in enumerate(seq) if (kind, what) == ("event", e)] for e in (la.START, la.STOP))
        assert len(a) == len(b) == 1, (name, seq)
        assert [k for _, k, _ in seq[a[0] + 1:b[0]]] == kernels, (name, op)


@pytest.mark.parametrize("dims,tiles,parts", [((21, 192, 64, 60, 25, 1, 1, 12), 6 * 2, 8), ((13, 64, 192, 69, 25, 1, 1, 12), 6 * 2, 8),
                                              ((3, 448, 64, 535, 17, 1, 1, 8), 14, 8), ((32, 768, 768, 800, 25, 1, 1, 12), 288 * 2, 3)], ids=str)
def test_parts_of_an_8_bit_weight_gradient(dims, tiles, parts):
    """Parts are waited for one after the other, eight at once: seven were chosen for the first three."""
    ((status, seq),) = la.run([{"call": "fp8_bwd", "dims": dims}])
    assert status == nm.NM_OK
    assert [grid[0] for _, kernel, grid in seq if kernel == "fp8_wgrad_kernel"] == [tiles * parts]


def test_batch_statistics_with_weights_at_any_address():
    """Weights at an address that is no multiple of 16 bytes, a view into a flat buffer, run on packed weights whatever the estimates
    say; the statistics then come from that engine's epilogue and not from a pass over its output."""
    d = (2, 256, 384, 240, 13, 1, 1, 6)
    (_, aligned), (_, odd) = la.run([{"call": "bn_fwd", "dims": d}, {"call": "bn_fwd", "dims": d, "w_offset": 2}])
    assert [k for _, k, _ in aligned][0] == "conv_unpacked_kernel"
    assert [k for _, k, _ in odd] == ["prepack_kernel", "conv_gemm_kernel", "bn_finalize_kernel", "bn_apply_fwd_kernel"]
