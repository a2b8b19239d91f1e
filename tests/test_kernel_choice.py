"""Which kernel a call runs on (host only): the layers of the encoder, calls of few tiles, rows of any length, float32."""
import pytest

from paper_1909_09577_amd import binding as nm
from paper_1909_09577_amd import inputs as syn

FWD, DGRAD, WGRAD, BN = nm.NM_OP_FWD, nm.NM_OP_BWD_DATA, nm.NM_OP_BWD_WEIGHT, nm.NM_OP_BN_FWD


def _align(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("cfg", [syn.JASPER_B1, syn.JASPER_B3, syn.EPILOG_A], ids=lambda c: c.name)
def test_full_size_layers_run_on_the_unrolled_kernels(cfg):
    for op in (FWD, DGRAD):
        assert nm.nm_conv1d_kernel_name(op, *cfg.dims()) == f"conv_gemm_kernel<5, 1, {cfg.K}, false, false, false, false>"
        assert nm.nm_conv1d_kernel_name(op, *cfg.dims(), masked=True) == f"conv_gemm_kernel<5, 1, {cfg.K}, true, false, false, false>"
    assert nm.nm_conv1d_kernel_name(BN, *cfg.dims()) == f"conv_gemm_kernel<5, 1, {cfg.K}, false, true, false, false>"
    assert nm.nm_conv1d_kernel_name(WGRAD, *cfg.dims()).startswith("wgrad_shared_kernel<")
    assert nm.nm_conv1d_kernel_name(FWD, *cfg.dims(), dtype=nm.NM_F32) == "f32_conv_kernel"
    assert nm.nm_conv1d_kernel_name(FWD, *cfg.dims(), flags=nm.NM_FORCE_DIRECT) == "direct_fwd_kernel"


def test_the_workspace_has_a_say():
    for K, engine, other in ((15, "conv_split_kernel<", 0), (25, "conv_unpacked_kernel<", 25)):
        few = (1, 768, 768, 600, K, 1, 1, K // 2)
        assert nm.nm_conv1d_kernel_name(FWD, *few).startswith(engine)
        full = nm.nm_conv1d_workspace_bytes(FWD, *few)
        # with less room fewer parts, without any the other engine
        least = -(-768 // 64) * (768 // 32) * (K + 1) * 256 * 16 + 512 * 16
        parts = [int(nm.nm_conv1d_kernel_name(FWD, *few, workspace_bytes=n).split(" in ")[1].split()[0]) for n in (full, least + (full - least) // 2)]
        assert parts[0] > parts[1] > 1
        assert nm.nm_conv1d_kernel_name(FWD, *few, workspace_bytes=least) == f"conv_gemm_kernel<5, 1, {other}, false, false, false, false>"
        with pytest.raises(nm.NmError) as e:
            nm.nm_conv1d_kernel_name(FWD, *few, workspace_bytes=least - 1)
        assert e.value.status == nm.NM_ERR_WORKSPACE
    odd = (16, 384, 384, 777, 13, 1, 1, 6)
    for op, plain in ((FWD, "direct_fwd_kernel"), (DGRAD, "direct_dgrad_kernel"), (WGRAD, "direct_wgrad_kernel")):
        assert not nm.nm_conv1d_kernel_name(op, *odd).startswith("direct")
        room = 0 if op == FWD else (2 * 16 * 384 * 777 + 255) // 256 * 256
        assert nm.nm_conv1d_kernel_name(op, *odd, workspace_bytes=room) == plain
    f32 = (4, 256, 256, 400, 11, 1, 1, 5)
    assert nm.nm_conv1d_kernel_name(WGRAD, *f32, dtype=nm.NM_F32) == "f32_wgrad_kernel"
    assert nm.nm_conv1d_kernel_name(WGRAD, *f32, dtype=nm.NM_F32, workspace_bytes=4 * 4 * 256 * 400) == "direct_wgrad_kernel"


def test_room_for_no_parts_is_not_taken_for_any_room():
    """The engine's plans are remembered by their limit: none must not be looked up as no limit."""
    dims = (7, 29, 640, 824, 7, 1, 1, 3)
    full = nm.nm_conv1d_workspace_bytes(DGRAD, *dims)
    least = _align((1 * 20 * 8 * 256 + 512) * 16) + _align(2 * 7 * 640 * 824)
    assert least < full
    for _ in range(2):
        name = nm.nm_conv1d_kernel_name(DGRAD, *dims, workspace_bytes=least)
        assert "conv_split" not in name or " in 1 parts" in name, name
        assert not nm.nm_conv1d_kernel_name(DGRAD, *dims).endswith(" in 1 parts")


def test_arguments_are_checked():
    import ctypes
    L = nm.lib()
    dims = (2, 64, 64, 64, 3, 1, 1, 1)
    name = ctypes.create_string_buffer(8)
    assert L.nm_conv1d_kernel_name(FWD, *dims, 0, 0, 0, 1 << 20, None, 8) == nm.NM_ERR_BAD_ARG
    assert L.nm_conv1d_kernel_name(FWD, *dims, 0, 0, 0, 1 << 20, name, 0) == nm.NM_ERR_BAD_ARG
    assert L.nm_conv1d_kernel_name(nm.NM_OP_BWD, *dims, 0, 0, 0, 1 << 20, name, 8) == nm.NM_ERR_BAD_ARG
    assert L.nm_conv1d_kernel_name(FWD, *dims[:4], 0, 1, 1, 1, 0, 0, 0, 1 << 20, name, 8) == nm.NM_ERR_BAD_ARG
    assert L.nm_conv1d_kernel_name(FWD, *dims, 0, 0, 0, 1 << 20, name, 8) == nm.NM_OK and len(name.value) == 7


@pytest.mark.parametrize("dims", [(32, 64, 256, 1600, 11, 5), (1, 64, 256, 320, 11, 5), (2, 384, 256, 112, 25, 12), (2, 64, 1024, 32, 3, 1),
                                  (8, 256, 128, 160, 12, 5), (4, 128, 64, 96, 2, 0)], ids=lambda d: "x".join(map(str, d)))
def test_stride2_gradient_in_the_workspace_of_one_contraction_per_parity(dims):
    """A workspace of the size that g, each parity's taps, its packed filter and its outputs take (what the call asked for
    while it made the parities one after the other) keeps the call on the matrix cores."""
    B, Cin, Cout, T, K, pad = dims
    To = nm.nm_conv1d_out_len(T, K, 2, 1, pad)
    assert T % 16 == 0 and To % 8 == 0
    room = _align(2 * B * Cout * To)
    for r in (0, 1):
        taps = (K - ((r + pad) & 1) + 1) // 2
        packed = _align((-(-Cin // 64) * -(-Cout // 32) * (taps + taps % 2) * 256 + 512) * 16)
        room += _align(2 * Cout * Cin * taps) + packed + _align(B * Cin * T)
    name = nm.nm_conv1d_kernel_name(DGRAD, B, Cin, Cout, T, K, 2, 1, pad, flags=nm.NM_RELU, workspace_bytes=room)
    assert not name.startswith("direct"), name


def test_parts_of_a_weight_gradient_where_their_sum_costs_more_than_they_save():
    """Few rows to add the parts up, few units to share out: eight parts are enough; the strided first layer takes more."""
    assert nm.nm_conv1d_kernel_name(WGRAD, 10, 64, 32, 560, 13, 1, 3, 18) == "wgrad_kernel<5> in 8 parts"
    assert nm.nm_conv1d_kernel_name(WGRAD, 6, 4, 256, 408, 13, 1, 3, 18) == "wgrad_kernel<5> in 8 parts"
    assert nm.nm_conv1d_kernel_name(WGRAD, 32, 64, 256, 1600, 11, 2, 1, 5) == "wgrad_kernel<6> in 16 parts"


@pytest.mark.parametrize("dtype", [nm.NM_BF16, nm.NM_F32], ids=["bf16", "f32"])
def test_the_smallest_calls_stay_on_the_plain_kernels(dtype):
    """A few products per thread are done before the matrix-core kernels' launches are; rows of 16-byte groups are as ever."""
    if dtype == nm.NM_BF16:
        assert nm.nm_conv1d_kernel_name(FWD, 3, 1, 512, 45, 1) == "direct_fwd_kernel"
        assert nm.nm_conv1d_kernel_name(DGRAD, 2, 45, 6, 20, 1) == "direct_dgrad_kernel"
        assert nm.nm_conv1d_kernel_name(DGRAD, 5, 37, 1, 13, 7, 2, 1, 3) == "direct_dgrad_kernel"
        assert not nm.nm_conv1d_kernel_name(FWD, 3, 16, 512, 45, 3, 1, 1, 1).startswith("direct")
        assert not nm.nm_conv1d_kernel_name(FWD, 3, 1, 512, 48, 1).startswith("direct")
    assert nm.nm_conv1d_kernel_name(WGRAD, 3, 421, 32, 23, 7, 2, 3, 9, dtype=dtype) == "direct_wgrad_kernel"
    assert not nm.nm_conv1d_kernel_name(WGRAD, 4, 256, 256, 401, 11, 1, 1, 5, dtype=dtype).startswith("direct")


def test_plans_in_parts_are_ranked_by_their_estimate():
    """Below the host's floor for a third launch all plans in parts cost the same against another engine; among themselves the
    first one tried (128-step tiles, four parts) must not win (K=13 on packed weights: 17.3 us on the device with 64-step tiles,
    19.1 with those).
    And a K=1 call whose other engine was estimated too high: 44 us there, 58 in the engine for few tiles."""
    assert nm.nm_conv1d_kernel_name(FWD, 1, 384, 384, 600, 12, 1, 1, 6).startswith("conv_split_kernel<2, 1>")
    assert nm.nm_conv1d_kernel_name(DGRAD, 23, 896, 64, 1496, 1) .startswith("pointwise_gemm_kernel<false")


def test_a_plan_in_one_part_is_no_way_out_of_a_small_workspace():
    """896 -> 16 channels, K=29: with the room of the weights alone the call goes to the other engine."""
    dims = (2, 896, 16, 304, 29, 1, 1, 14)
    least = (1 * 28 * 30 * 256 + 512) * 16
    assert least < nm.nm_conv1d_workspace_bytes(FWD, *dims)
    assert nm.nm_conv1d_kernel_name(FWD, *dims, workspace_bytes=least).startswith("conv_gemm_kernel<")
    assert nm.nm_conv1d_kernel_name(FWD, *dims).startswith("conv_split_kernel<")


def test_smallest_calls_run_on_the_plain_kernels():
    assert nm.nm_conv1d_kernel_name(FWD, 9, 16, 64, 68, 1) == "direct_fwd_kernel"
    assert nm.nm_conv1d_kernel_name(WGRAD, 7, 256, 16, 47, 21, 3, 1, 10, dtype=nm.NM_F32) == "direct_wgrad_kernel"
    assert nm.nm_conv1d_kernel_name(FWD, 4, 256, 256, 400, 11, 1, 1, 5) != "direct_fwd_kernel"
