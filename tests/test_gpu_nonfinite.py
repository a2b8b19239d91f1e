"""Infinities: the matrix-core kernels multiply zeros for the padding, behind a row and for absent taps.  In float32 and on rows
of any length, which plain kernels without such products served before them, one infinite sample or gradient must leave finite
what the definition leaves finite (in float32 one infinite weight too): results are finite where the plain kernels' are, at the
usual gates."""
import pytest

from oracle import conv1d_oracle as orc
from paper_1909_09577_amd import binding as nm

pytestmark = pytest.mark.gpu

# (dtype, B, Cin, Cout, T, K, stride, dilation, pad), kernel of the forward pass
CASES = {
    ("f32", 2, 40, 72, 130, 11, 1, 1, 5): "f32_conv",
    ("f32", 2, 24, 40, 201, 5, 2, 1, 2): "f32_conv",
    ("f32", 1, 24, 80, 100, 32, 1, 1, 16): "f32_conv",
    ("bf16", 2, 64, 96, 133, 11, 1, 1, 5): "conv_split_kernel<2, 1> in 1 parts",
    ("bf16", 1, 512, 64, 133, 9, 1, 2, 8): "conv_split_kernel<2, 1> in 16 parts",
    ("bf16", 1, 256, 256, 133, 11, 1, 1, 5): "conv_unpacked_kernel<2, 11, false>",
    ("bf16", 1, 512, 512, 131, 25, 1, 1, 12): "conv_unpacked_kernel<2, 25, false>",
    ("bf16", 1, 256, 256, 133, 13, 1, 2, 12): "conv_unpacked_kernel<2, 13, false>",
    ("bf16", 20, 128, 512, 1277, 11, 1, 1, 5): "conv_gemm_kernel<5, 1, 11, true, false, true",        # the unrolled kernel
    ("bf16", 8, 256, 200, 801, 7, 1, 1, 3): "conv_gemm_kernel<5, 1, 0, false, false, true, false>",    # tap pairs, an absent eighth tap
    ("bf16", 8, 256, 200, 798, 7, 1, 1, 4): "conv_gemm_kernel<5, 1, 0, false, false, true, false>",    # the same, only the input rows odd
    ("bf16", 8, 480, 250, 801, 5, 1, 1, 2): "conv_gemm_kernel<5, 1, 0, false, false, true, true>",     # the same with a pad pair
    ("bf16", 8, 256, 1024, 1277, 1, 1, 1, 0): "pointwise_gemm_kernel<true",
    ("bf16", 3, 64, 128, 175, 4, 1, 1, 2): "conv_split_kernel<2, 1>",                                 # only the input rows are odd
    ("bf16", 3, 40, 72, 123, 11, 2, 1, 5): "conv_split_kernel<2, 2>",  # parities of a stride-2 gradient: filters of five and six taps
    ("bf16", 3, 40, 72, 160, 11, 2, 1, 5): "conv_split_kernel<2, 2>",  # the same on 16-byte rows (its gradient only)
}


def _same(got, ref, dtype, what):
    import torch
    got, ref = got.double(), ref.double()
    ok = ref.isfinite()
    assert torch.equal(got.isfinite(), ok), f"{what}: {int((~got.isfinite()).sum())} not finite, plain kernels {int((~ok).sum())}"
    rms = ref[ok].square().mean().sqrt()
    # two results within the gate of the other parity tests, so within twice the gate of each other
    assert ((got - ref)[ok].abs() / (ref[ok].abs() + rms)).max() <= (2e-2 if dtype == "bf16" else 2e-5), what
    assert ok.any() and not ok.all(), f"{what}: the case shows nothing"


@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_one_infinite_element(case, masked):
    import torch
    dtype, B, Cin, Cout, T, K, stride, dil, pad = case
    name = nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *case[1:], dtype=nm.NM_F32 if dtype == "f32" else nm.NM_BF16, masked=masked)
    assert name.startswith(CASES[case]), name
    if "conv_unpacked" in name:  # the gradient's infinities go through the flipped instance
        back = nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_DATA, *case[1:], masked=masked)
        assert back.startswith(f"conv_unpacked_kernel<2, {case[5]}, true>"), back
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    To = orc.out_len(T, K, stride, dil, pad)
    kw = dict(stride=stride, dilation=dil, pad=pad)
    if masked:
        kw["lengths"] = torch.tensor([T - 3 * b for b in range(B)], dtype=torch.int32, device="cuda").clamp_min(T // 2)
    gen = torch.Generator(device="cuda").manual_seed(3)

    def randn(*shape):
        v = torch.randn(*shape, device="cuda", generator=gen)
        return torch.where(v == 0, 1, v).to(dt)

    x, w, dy = randn(B, Cin, T), randn(Cout, Cin, K) / (Cin * K) ** 0.5, randn(B, Cout, To)
    scale = torch.rand(Cout, device="cuda", generator=gen) + 0.5

    def with_inf(t, *at):
        t = t.clone()
        t[at] = float("inf")
        return t

    last = int(kw["lengths"][0]) - 1 if masked else T - 1  # the last valid sample of item 0
    rows16 = T % 8 == 0 and To % 8 == 0 and dtype == "bf16"
    for what, xi, wi, gi in [("x start", with_inf(x, 0, 1, 0), w, dy), ("x end", with_inf(x, 0, 1, last), w, dy), ("w", x, with_inf(w, 1, 1, K // 4), dy),
                             ("dy start", x, w, with_inf(dy, 0, 1, 0)), ("dy end", x, w, with_inf(dy, 0, 1, To - 1))]:
        def passes(direct):
            c = dict(kw, force_direct=direct)
            return (nm.nm_conv1d_block_fwd(xi, wi, scale, None, None, **c), nm.nm_conv1d_bwd_data(gi, wi, T, scale=scale, **c)[0],
                    nm.nm_conv1d_bwd_weight(xi, gi, K, scale=scale, **c), *nm.nm_conv1d_bwd(xi, gi, wi, scale=scale, **c)[::2])
        (y, dx, dw, dx2, dw2), (yr, dxr, dwr, _, _) = passes(False), passes(True)
        assert torch.equal(dx2.isnan(), dx.isnan()) and torch.equal(dw2.isnan(), dw.isnan())
        in_x, in_w, in_g = what.startswith("x"), what == "w", what.startswith("dy")
        if not rows16 and (in_x or (in_w and dtype == "f32")):
            _same(y, yr, dtype, f"y, {what}")
        if in_g or (in_w and dtype == "f32"):
            _same(dx, dxr, dtype, f"dx, {what}")
        if not rows16 and (in_x or in_g):
            _same(dw, dwr, dtype, f"dw, {what}")
