"""Which kernel a convolution runs on, at the lines between kernels: the names
that libctc.so gives need no GPU.  What the kernels compute there is the GPU
tests' matter."""
import pytest

ctc = pytest.importorskip("paper_2609_16742_amd.ctc")


def _name(dtype, n, h, w, c_in, c_out, k, stride=1):
    d = ctc.layer_desc(c_in, c_out, k, k, stride, k // 2, 1, 1, ctc.CTC_ROLE_SUM)
    return ctc.ctc_conv2d_kernel_name(d, ctc.DTYPES[dtype], n, h, w)


# layer, whether conv_lat (one wave per 16 x 16 output tile) is the faster kernel
LAT = [
    # pointwise: conv_pw up to 64 (48) channels
    (("f16", 2, 63, 63, 16, 16, 1), False), (("f16", 13, 19, 15, 32, 32, 1), False),
    (("f16", 1, 28, 28, 64, 64, 1), False), (("f16", 1, 28, 28, 64, 72, 1), True),
    (("f16", 1, 14, 14, 160, 48, 1), False), (("f16", 1, 14, 14, 160, 56, 1), True),
    (("f16", 1, 14, 14, 32, 256, 1), False), (("f16", 1, 14, 14, 96, 512, 1), True),
    # few steps of k
    (("f16", 1, 72, 72, 16, 24, 3), False), (("f16", 1, 72, 72, 24, 24, 3), True),
    (("f16", 2, 36, 36, 144, 96, 1, 2), True), (("f16", 1, 28, 28, 144, 168, 1, 2), False),
    (("f16", 1, 14, 14, 96, 576, 1), False), (("f16", 1, 14, 14, 392, 576, 1), True),
    (("f32", 1, 14, 14, 36, 96, 1), False), (("f32", 1, 14, 14, 68, 96, 1), True),
    # one wave per SIMD and more of them
    (("f16", 4, 14, 14, 264, 264, 3), True), (("f16", 5, 14, 14, 264, 264, 3), False),
    (("f16", 4, 28, 28, 128, 128, 3), True), (("f16", 1, 28, 28, 512, 512, 3), True),
    (("f32", 4, 14, 14, 260, 260, 3), True), (("f32", 5, 14, 14, 260, 260, 3), False),
    (("f32", 8, 14, 14, 256, 256, 3), True), (("f32", 12, 28, 28, 36, 40, 3), True),
    # up to 32 channels: whole input in an L2, in none, past them all
    (("f16", 4, 56, 56, 72, 32, 3), True), (("f16", 4, 56, 56, 264, 32, 3), False),
    (("f16", 19, 49, 49, 664, 32, 3, 2), True), (("f16", 4, 56, 56, 264, 16, 3), True),
]


@pytest.mark.parametrize("layer,lat", LAT)
def test_small_layers_take_the_faster_kernel(layer, lat):
    assert _name(*layer).startswith("conv_lat") == lat, _name(*layer)


# layer, its kernel: the lines between conv_pp's tiles, which are its rounds of
# workgroups
TILES = [
    # 256 tiles of 128 x 128 (two 128 x 64 tiles per CU), one more pixel tile
    (("f16", 1, 128, 128, 128, 256, 3), "conv_pp<128, 64, 0, false>"),
    (("f16", 1, 128, 129, 128, 256, 3), "conv_pp<128, 96, 0, false>"),
    (("f16", 1, 128, 128, 136, 248, 3), "conv_ppr<_Float16, 128, 64>"),
    (("f16", 1, 128, 129, 136, 248, 3), "conv_ppr<_Float16, 128, 128>"),
    # 64 x 96 tiles: 510 (512), 684 (680), 768, 771, 1026 (1024) of them
    (("f16", 1, 96, 170, 264, 168, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 171, 264, 168, 3), "conv_dma<_Float16, 128, 64, 2, 2, 2, true, 0, false, 0>"),
    (("f16", 1, 96, 171, 104, 168, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 228, 264, 168, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 256, 264, 168, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 257, 264, 168, 3), "conv_ppr<_Float16, 128, 128>"),
    (("f16", 1, 96, 768, 136, 64, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 769, 136, 64, 3), "conv_dma<_Float16, 128, 64, 2, 2, 2, true, 0, false, 0>"),
    (("f16", 1, 96, 769, 264, 64, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 1, 96, 1025, 136, 64, 3), "conv_ppr<_Float16, 64, 96>"),
    # filters in registers: 3072 strip rows, 4608 up to 32 channels
    (("f16", 54, 28, 28, 64, 40, 3), "conv_ppr<_Float16, 64, 96>"),
    (("f16", 55, 28, 28, 64, 40, 3), "conv_rows<false, true, false>"),
    (("f16", 82, 28, 28, 64, 32, 3), "conv_dma<_Float16, 64, 32, 4, 1, 2, true, 0, false, 0>"),
    (("f16", 83, 28, 28, 64, 32, 3), "conv_rows<false, true, false>"),
    (("f16", 14, 56, 56, 64, 32, 3), "conv_rows<false, true, false>"),
]


@pytest.mark.parametrize("layer,name", TILES)
def test_layers_take_the_tile_of_their_rounds(layer, name):
    assert _name(*layer) == name
