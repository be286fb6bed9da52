"""Which kernel a 3x3 / stride 1 layer runs on where the estimates of two are close (host-only; the times are beside the rules)."""
import pytest

from paper_1904_08368_amd import binding as B

F16, I8 = B.RELAY_F16, B.RELAY_I8
HALO128 = ("conv3x3_halo_kernel<true, 2, 2, 2, 1,", "conv3x3_halo_kernel<false, 2, 2, 2, 1,")
IGEMM = ("igemm_dma_kernel<",)


# layers that 128 x 64 tiles suit stay there unless another kernel is clearly faster; tiles too large for a CU's LDS
@pytest.mark.parametrize("dtype,n,c,h,w,k,kernels", [
    (I8, 42, 576, 27, 13, 80, HALO128), (I8, 11, 576, 71, 41, 40, HALO128), (I8, 3, 192, 170, 7, 464, HALO128), (F16, 54, 160, 36, 8, 96, HALO128),
    (F16, 35, 416, 145, 15, 24, HALO128), (F16, 7, 352, 112, 30, 152, HALO128),
    (F16, 8, 64, 65, 126, 16, IGEMM), (F16, 34, 64, 23, 121, 56, IGEMM), (I8, 44, 128, 18, 72, 64, IGEMM), (I8, 1, 128, 151, 77, 296, IGEMM),
    (I8, 3, 128, 175, 68, 32, ("conv3x3_halo_kernel<true, 2, 2, 1, 1, 2,",)),
    (F16, 32, 256, 56, 56, 256, ("conv3x3_halo_kernel<false, 4, 2, 2, 2, 2,",)), (F16, 32, 64, 224, 224, 64, ("conv3x3_halo_kernel<false, 4, 1, 2, 2, 2, 2, true",))])
def test_choice(dtype, n, c, h, w, k, kernels):
    d = B.conv_desc(n, c, h, w, k, 3, 3, 1, 1, dtype, B.RELAY_NHWC, 0)
    name = B.relay_conv2d_kernel_name(d)
    assert name.startswith(kernels), name


@pytest.mark.parametrize("n,h,w,kernel", [(31, 57, 37, "igemm_dma_kernel"), (20, 56, 59, "conv3x3_halo_kernel<false, 4, 1"), (32, 56, 56, "conv3x3_halo_kernel<false, 4, 1"),
                                          (18, 57, 59, "conv3x3_halo_kernel<false, 2, 2")])
def test_64_channels_around_one_round_of_slots(n, h, w, kernel):
    """Tiles of 128 pixels without and with the pad positions of the 3x3 kernel: 511 / 534, 517 / 535, 784 / 813, 473 / 490."""
    d = B.conv_desc(n, 64, h, w, 64, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, 0)
    assert B.relay_conv2d_kernel_name(d).startswith(kernel)
