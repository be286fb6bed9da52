"""The one-launch depthwise + 1x1 kernel for layers of few pixels, against the oracle's two fused operators and bit for bit
against the two separate launches: every variant at the edges of its tiles, and the rule that chooses them."""
import ctypes as C

import pytest
import torch

from tests.test_gpu_dwpw import _case

# (most channels, ring stages of 32 channels) of every variant, in the library's order
VARIANTS = ((256, 8), (256, 8), (256, 8), (1024, 32), (512, 16), (512, 16), (512, 8), (512, 6), (512, 4))


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


@pytest.mark.gpu
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("variant", range(len(VARIANTS)))
def test_every_variant_at_the_edges(G, variant, stride):
    """Images narrower and wider than a rectangle, odd and even, a single pixel, channel tiles that end within a wave's
    32 channels, the fewest channels and the most, one image and several."""
    most = VARIANTS[variant][0]
    for i, (n, c, h, w, k) in enumerate([(1, 32, 1, 1, 8), (2, 64, 5, 3, 40), (1, most, 7, 7, 264), (3, 64, 9, 33, 72), (1, 128, 2, 70, 136),
                                         (1, most // 2, 14, 15, 64)]):
        _case(G, 9000 + 100 * variant + 10 * stride + i, n, c, h, w, k, stride, variant=200 + variant, plain_tail=i % 2 == 1)


def test_a_forced_variant_that_does_not_take_the_shape_is_an_error():
    """(host only: every check runs before the first launch)"""
    from paper_1904_08368_amd import binding as B
    d = B.conv_desc(1, 384, 14, 14, 384, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, 0)     # no power of two of channels
    assert "direct" not in B.relay_dwconv_pwconv_kernel_name(d, 512)
    mem = [(1 << 30) + i * 4096 for i in range(4)]
    for tile in (500, 508, 300):
        B.relay_set_conv_tile(tile)
        try:
            if tile == 300:
                d = B.conv_desc(1, 384, 14, 14, 384, 3, 3, 2, 1, B.RELAY_F16, B.RELAY_NHWC, 0)     # a variant for stride 1
            with pytest.raises(B.RelayError) as e:
                B.relay_dwconv_pwconv_kernel_name(d, 512)
            assert e.value.status == 4
            assert B.lib().relay_fused_dwconv_pwconv(C.byref(d), mem[0], mem[1], None, None, None, 512, 0, mem[2], None, None, None, mem[3], None) == 4
        finally:
            B.relay_set_conv_tile(-1)


# the first and last sizes at which the rule takes a tile (the number of workgroups that fit the chip at once)
@pytest.mark.gpu
@pytest.mark.parametrize("n,c,h,w,k,stride,name", [
    (1, 64, 32, 32, 64, 1, "16, 2, 4, 8, 8, 0, 2"), (8, 64, 28, 28, 64, 1, "32, 4, 4, 8, 8, 0, 2"), (2, 512, 14, 14, 512, 1, "16, 2, 8, 16, 16, 0, 2"), (1, 1024, 7, 7, 1024, 1, "16, 1, 8, 32, 32, 0, 2"),
    (1, 512, 14, 14, 256, 1, "16, 1, 8, 32, 32, 0, 2"), (4, 512, 14, 14, 512, 1, "32, 2, 8, 16, 16, 0, 2"), (32, 512, 14, 14, 512, 1, "64, 8, 8, 4, 16, 2, 4"),
    (37, 512, 14, 14, 512, 1, None), (3, 1024, 7, 7, 1024, 1, None), (1, 32, 16, 16, 64, 1, None)])
def test_rule(G, n, c, h, w, k, stride, name):
    from paper_1904_08368_amd import binding as B
    d = B.conv_desc(n, c, h, w, c, 3, 3, stride, 1, B.RELAY_F16, B.RELAY_NHWC, 0)
    got = B.relay_dwconv_pwconv_kernel_name(d, k)
    assert (f"dwpw_fused_direct_kernel<{stride}, {name}>" == got) if name else ("direct" not in got)
    assert B.relay_dwconv_pwconv_few_pixels(d, k) == (name is not None)


# most channels of the variants with items of four rows (9 to 11) or three workgroups to a CU (11, 12)
@pytest.mark.gpu
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("variant,most", [(9, 512), (10, 512), (11, 128), (12, 128)])
def test_variants_of_one_item_in_registers_at_the_edges(G, variant, most, stride):
    """Heights of every remainder of four, images lower than an item, rectangles that end past the image, channel tiles that
    end within a wave's 32 channels, threads without an item, several rounds of workgroups."""
    for i, (n, c, h, w, k) in enumerate([(1, 32, 1, 1, 8), (2, 64, 5, 3, 40), (1, most, 7, 7, 136), (3, 64, 9, 33, 72), (1, 128, 2, 70, 136),
                                         (1, most // 2, 14, 15, 64), (2, most, 11, 13, 128), (1, most, 10, 6, 8), (5, 128, 60, 61, 128)]):
        _case(G, 9900 + 100 * variant + 10 * stride + i, n, c, h, w, k, stride, variant=200 + variant, plain_tail=i % 2 == 1)


@pytest.mark.gpu
@pytest.mark.parametrize("n,c,h,w,k,stride,name", [
    (32, 64, 56, 56, 64, 1, "64, 4, 4, 4, 4, 3, 2"), (32, 64, 56, 56, 136, 1, None), (32, 128, 56, 56, 128, 1, "64, 4, 4, 4, 4, 3, 4"),
    (32, 128, 56, 56, 128, 2, "64, 4, 4, 4, 4, 3, 2"), (7, 128, 90, 70, 128, 2, "64, 8, 8, 4, 16, 0, 2"), (32, 512, 10, 9, 512, 1, "32, 8, 8, 6, 16, 0, 2"),
    (32, 256, 18, 18, 256, 1, "64, 8, 8, 4, 16, 2, 4"), (32, 256, 56, 56, 256, 1, None)])
def test_rule_beyond_one_round(G, n, c, h, w, k, stride, name):
    test_rule(G, n, c, h, w, k, stride, name)
