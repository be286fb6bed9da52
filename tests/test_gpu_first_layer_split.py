"""The first-layer conv2d where its output channels are spread over workgroups: 16 a workgroup, and the sizes on both sides
(8 a workgroup, all of them), against the CPU oracle."""
import pytest
import torch

import oracle as O
from tests.test_gpu_first_layer import TOL_F16, _case

pytestmark = pytest.mark.gpu


# waves of pixel threads x groups of 16 channels: at most 256 -> 8 channels, more -> 16, a single group or above 1600 waves -> all
@pytest.mark.parametrize("shape", [(1, 128, 256, 128), (1, 130, 256, 128), (2, 224, 224, 48), (3, 224, 224, 16), (17, 224, 224, 32)])
def test_channel_groups(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as G
    n, h, w, k = shape
    x, wt, b, sc, sf = _case(h + k + n, n, h, w, k)
    want = O.fused_conv2d(x, wt, stride=(2, 2), pad=(1, 1), bias=b, scale=sc, shift=sf, relu_flag=True, out_dtype="f16")
    got = G.run_first_layer_f16(x, wt, bias=b, scale=sc, shift=sf, relu=True)
    assert O.max_rel_err(got, want) <= TOL_F16
