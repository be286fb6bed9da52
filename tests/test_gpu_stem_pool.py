"""The pooled first layer that stages its input patch once (padded NHWC4 image, stride 2): against the oracle and bit for bit
against the two separate calls, over filter sizes, channel counts, ragged channel tiles and several blocks in both directions."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.test_gpu_convpool import TOL_F16, _oracle_f16
from workloads import inputs, nets

pytestmark = pytest.mark.gpu

# (n, c, h, w, k, r): stride 2, conv outputs of 14 a x 16 b; the last has the most filter rows the form does not take
CASES = [(2, 3, 28, 32, 64, 7), (1, 3, 56, 96, 72, 7), (3, 4, 28, 64, 136, 5), (2, 1, 56, 32, 8, 3), (1, 2, 84, 32, 40, 1), (1, 3, 28, 32, 16, 8)]


@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_stem_pool(case, i8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    from tests import gpu_util as G
    n, c, h, w, k, r = case
    pd = (r - 1) // 2
    g = np.random.default_rng(inputs.BASE_SEED + 98000 + r * 10 + c)
    d = B.conv_desc(n, c, h, w, k, r, r, 2, pd, B.RELAY_I8 if i8 else B.RELAY_F16, B.RELAY_NHWC4_PADDED, 0)
    assert B.relay_conv2d_maxpool_fusable(d)
    assert (", 1, 1, 1, false" in B.relay_conv2d_maxpool_kernel_name(d)) == (r <= 7)
    if i8:
        x = g.integers(-127, 128, (n, c, h, w)).astype(np.int8)
        wt = g.integers(-127, 128, (k, c, r, r)).astype(np.int8)
        b = g.integers(-2000, 2000, k).astype(np.int32)
        want = O.maxpool2d(O.qconv2d_requant(x, wt, stride=(2, 2), pad=(pd, pd), bias=b, out_rshift=9, relu_flag=False), 3, 2, 1).astype(np.int8)
        got = G.run_qconv_pool(x, wt, 2, pd, bias=b, rshift=9)
        assert np.array_equal(got, want)
        if k % 16 == 0:   # (what the int8 pool by itself takes)
            assert np.array_equal(got, G.run_qconv_pool(x, wt, 2, pd, bias=b, rshift=9, fused=False))
    else:
        op = nets.conv("c", "x", "y", c, k, r, 2, pd, bias=True, bn=True, relu=False)
        p = inputs.layer_params(op, 33, k + r, "f16")
        x = inputs.activation(33, c + h, (n, c, h, w), "f16")
        got = G.run_conv_pool_f16(x, p["w"], 2, pd, bias=p["bias"], scale=p["scale"], shift=p["shift"])
        two = G.run_conv_pool_f16(x, p["w"], 2, pd, bias=p["bias"], scale=p["scale"], shift=p["shift"], fused=False)
        assert O.max_rel_err(got, _oracle_f16(x, p, 2, pd, False)) <= TOL_F16
        assert np.array_equal(got.view(np.uint16), two.view(np.uint16))
