"""Pointwise layers of whole tiles: the engine that was measured to be the faster one, and the others' calls where they were."""
import pytest

from paper_1909_09577_amd import binding as nm


@pytest.mark.parametrize("dims,kernel", [((1, 512, 640, 600), "conv_split_kernel<2, 1> in 2 parts"), ((1, 896, 1024, 56), "conv_split_kernel<2, 1> in"),
                                         ((3, 384, 512, 117), "conv_split_kernel"), ((16, 768, 768, 800), "pointwise_gemm_kernel<false, 2, 5, 128>"),
                                         ((32, 896, 1024, 800), "pointwise_gemm_kernel<false, 4, 4, 64>"),
                                         ((23, 64, 896, 1496), "pointwise_gemm_kernel"), ((2, 502, 302, 176), "pointwise_gemm_kernel<false, 2, 5, 128>"),
                                         ((1, 1024, 29, 97), "decoder_mfma_kernel<true, true, 4>"), ((1, 1024, 29, 96), "decoder_mfma_kernel<true, false, 4>")], ids=str)
def test_choice(dims, kernel):
    assert nm.nm_conv1d_kernel_name(nm.NM_OP_FWD, *dims, 1, 1, 1, 0, flags=nm.NM_RELU).startswith(kernel)
