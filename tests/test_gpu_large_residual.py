"""A 3x3 conv whose residual and output are larger than 2^31 bytes: the 3x3 kernel addresses the residual with 32-bit byte offsets,
unsigned, and marks lanes without a pixel by the offset 2^31, which here lies inside the tensor.  Against fp32 on the CPU at the
first and last rows of the images, where such lanes are, and on both sides of the 2^31st byte."""
import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


def test_residual_and_output_beyond_two_gib(G):
    from paper_1904_08368_amd import binding as B
    n, c, h, w, k = 9, 64, 481, 487, 520      # (the 2^31st byte lies in row 392 of the last image)
    d = B.conv_desc(n, c, h, w, k, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(None, True, True, True))
    assert (1 << 31) < n * h * w * k * 2 < (1 << 32)
    assert "conv3x3_halo_kernel" in B.relay_conv2d_kernel_name(d)
    g = torch.Generator(device=G.DEV).manual_seed(41)
    x = torch.randn((n, h, w, c), generator=g, device=G.DEV).half()
    res = torch.randn((n, h, w, k), generator=g, device=G.DEV, dtype=torch.float16)
    wsrc = (torch.randn((k, c, 3, 3), generator=g, device=G.DEV) * (2 / (9 * c)) ** 0.5).half()
    scale, shift = (1 + 0.1 * torch.randn(k, generator=g, device=G.DEV)), 0.1 * torch.randn(k, generator=g, device=G.DEV)
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, wsrc, c, wp)
    y = torch.full((n, h, w, k), float("nan"), dtype=torch.float16, device=G.DEV)
    B.relay_fused_conv2d_bias_bn_relu(d, x, wp, None, scale, shift, res, y, None)
    torch.cuda.synchronize()
    edge = ((1 << 31) // (2 * k) - (n - 1) * h * w) // w     # the row of the last image that holds the 2^31st byte
    assert 4 < edge < h - 4
    wf, sc, sf = wsrc.float().cpu(), scale.cpu(), shift.cpu()
    for img, r0, r1 in ((0, 0, 2), (n - 2, h - 2, h), (n - 1, 0, 2), (n - 1, edge - 2, edge + 3), (n - 1, h - 3, h)):
        lo, hi = max(r0 - 1, 0), min(r1 + 1, h)
        rows = F.pad(x[img, lo:hi].float().cpu().permute(2, 0, 1)[None], (1, 1, int(r0 == 0), int(r1 == h)))
        want = F.conv2d(rows, wf)[0].permute(1, 2, 0) * sc + sf + res[img, r0:r1].float().cpu()
        got = y[img, r0:r1].float().cpu()
        # (one rounding of the result to fp16, 2^-11 of it, beside fp32 sums of 576 products)
        assert torch.allclose(got, want.relu(), rtol=2 ** -11 * 1.05, atol=2e-5), (img, r0, (got - want.relu()).abs().max())
    # no row anywhere was left out
    for img in range(n):
        assert not torch.isnan(y[img].float().sum())
