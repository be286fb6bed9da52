"""Which layers a forced split of the reduction takes off the 3x3 kernel (host-only: names and workspace sizes)."""
import pytest

from paper_1904_08368_amd import binding as B


def _d(dtype, n, c, h, k):
    return B.conv_desc(n, c, h, h, k, 3, 3, 1, 1, dtype, B.RELAY_NHWC, B.RELU)


def _under(split, d):
    B.relay_set_conv_split(split)
    try:
        return B.relay_conv2d_kernel_name(d), B.relay_workspace_bytes(d)
    finally:
        B.relay_set_conv_split(0)


F16, I8 = B.RELAY_F16, B.RELAY_I8
# a full chip of 128 x 64 tiles or several
WHOLE = [(F16, 32, 256, 56, 256), (F16, 32, 64, 56, 64), (F16, 32, 128, 28, 128), (F16, 32, 512, 14, 512), (F16, 8, 256, 28, 256),
         (F16, 32, 512, 7, 512), (I8, 16, 64, 56, 64), (I8, 16, 128, 28, 128)]
# too few tiles, or more than the 3x3 kernel's range
SPLIT = [(F16, 8, 512, 14, 512), (F16, 1, 256, 14, 256), (I8, 8, 512, 14, 512), (F16, 32, 128, 112, 128)]


@pytest.mark.parametrize("layer", WHOLE + SPLIT)
def test_never_split_is_the_kernel_of_the_shape(layer):
    d = _d(*layer)
    name, ws = _under(1, d)
    assert ws == 0
    if B.relay_conv2d_kernel_name(d).startswith("conv3x3_halo_kernel"):
        assert name == B.relay_conv2d_kernel_name(d)


@pytest.mark.parametrize("split", [2, 36])
@pytest.mark.parametrize("layer", WHOLE)
def test_layers_that_stay_whole(layer, split):
    d = _d(*layer)
    name = B.relay_conv2d_kernel_name(d)
    assert name.startswith("conv3x3_halo_kernel")
    assert _under(split, d) == (name, 0)


@pytest.mark.parametrize("layer", SPLIT)
def test_layers_that_are_split(layer):
    name, ws = _under(2, _d(*layer))
    assert name.startswith("igemm_dma_kernel") and ws > 0
