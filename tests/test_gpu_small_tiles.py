"""GPU parity of the kernel for layers of few output tiles (its waves split a tile's reduction): every tile shape at
ragged pixel and channel counts, reductions shorter than the number of waves and longer than the ring, one to four
steps per unit, strides, borders and the residual operand, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu
# Both sides round to fp16.  Where the fp32 sums (of at most 4608 products of unit-scale data, under 1e-5 of the
# result's scale from the exact ones) lie on the other side of a rounding boundary the two are one unit in the last
# place apart: at most 2^-10 of the value.
TOL_F16 = 2.0 ** -10 + 1e-5
VARIANTS = range(400, 406)

# n, c, h, w, k, r, stride, pad
SHAPES = [
    (1, 32, 5, 7, 24, 1, 1, 0),      # one step: every wave but the first is idle
    (2, 64, 9, 5, 72, 3, 1, 1),      # ragged pixels and channels, all four borders
    (1, 96, 7, 7, 20, 3, 2, 1),      # odd number of steps per tap, channels not a multiple of 8
    (3, 128, 6, 4, 40, 3, 1, 1),     # four steps per unit
    (1, 512, 4, 4, 64, 3, 1, 1),     # a long reduction: the ring wraps many times
    (1, 64, 11, 13, 16, 5, 2, 2),    # a wider window
    (1, 3, 21, 17, 16, 7, 2, 3),     # row-packed first layer
]


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("tile", VARIANTS)
@pytest.mark.parametrize("shape", SHAPES)
def test_fp16_small_tiles_match_the_oracle(G, shape, tile):
    n, c, h, w, k, r, s, p = shape
    g = np.random.default_rng(8100 + c + tile)
    x = g.standard_normal((n, c, h, w)).astype(np.float16)
    wt = (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
    ho, wo = (h + 2 * p - r) // s + 1, (w + 2 * p - r) // s + 1
    res = g.standard_normal((n, k, ho, wo)).astype(np.float16) if k % 8 == 0 else None
    b, sc, sf = (g.standard_normal(k).astype(np.float32) for _ in range(3))
    want = O.fused_conv2d(x, wt, stride=(s, s), pad=(p, p), bias=b, scale=sc, shift=sf, residual=res, relu_flag=True,
                          out_dtype="f16")
    got = G.run_conv_f16(x, wt, s, p, bias=b, scale=sc, shift=sf, residual=res, relu=True, tile=tile)
    assert O.max_rel_err(got, want) <= TOL_F16


@pytest.mark.parametrize("tile", VARIANTS)
@pytest.mark.parametrize("shape", [(n, c if c == 3 else c * 2, h, w, k, r, s, p) for n, c, h, w, k, r, s, p in SHAPES])
def test_int8_small_tiles_are_bit_exact(G, shape, tile):
    n, c, h, w, k, r, s, p = shape
    g = np.random.default_rng(8200 + c + tile)
    x = g.integers(-127, 128, (n, c, h, w)).astype(np.int8)
    wt = g.integers(-127, 128, (k, c, r, r)).astype(np.int8)
    ho, wo = (h + 2 * p - r) // s + 1, (w + 2 * p - r) // s + 1
    res = g.integers(-127, 128, (n, k, ho, wo)).astype(np.int8) if k % 16 == 0 else None
    bias = g.integers(-5000, 5000, k).astype(np.int32)
    want = O.qconv2d_requant(x, wt, stride=(s, s), pad=(p, p), bias=bias, residual=res, residual_lshift=6, out_rshift=12,
                             relu_flag=False)
    got = G.run_qconv(x, wt, s, p, bias=bias, residual=res, lshift=6, rshift=12, tile=tile)
    assert np.array_equal(got, want)


def test_segments_are_stored_where_they_belong(G):
    """Three members of a combined launch on small tiles: channel ranges of wider tensors on both sides."""
    from tests.test_gpu_combine import _check_members, _members, _run_combined
    from paper_1904_08368_amd import binding as B
    from workloads import inputs
    ops, params = _members(64, (8, 24, 40), 3, 1, bias=True)
    x = inputs.activation(21, 1, (1, 64, 9, 7), "f16")
    assert "igemm_small_kernel" in B.relay_conv2d_kernel_name(
        B.conv_desc(1, 64, 9, 7, 72, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, B.HAS_BIAS | B.HAS_BN | B.RELU))
    plan = [(0, 16, 64), (1, 0, 24), (0, 24, 64)]
    outs, bufs = _run_combined(G, x, ops, params, 1, 1, True, x_wide=96, x_off=32, out_plan=plan)
    _check_members(x, ops, params, outs, 1, 1, True)
    assert torch.all(bufs[0][..., :16] == -77.0)


def test_the_library_takes_small_tiles_at_batch_1_only(G):
    from paper_1904_08368_amd import binding as B
    d = lambda n, c, hw, k, r: B.conv_desc(n, c, hw, hw, k, r, r, 1, r // 2, B.RELAY_F16, B.RELAY_NHWC, B.RELU)
    for c, hw in ((64, 56), (128, 28), (256, 14), (512, 7)):
        assert "igemm_small_kernel" in B.relay_conv2d_kernel_name(d(1, c, hw, c, 3))
        assert "igemm_small_kernel" not in B.relay_conv2d_kernel_name(d(32, c, hw, c, 3))


# The rounding error of the fp32 sums themselves: every pixel alike, so that one shift per channel takes the exact result off
# at all of them, and what is left, scaled into fp16's range, is the error of the sum.
SCALE = 2.0 ** 14


def _sum_errors(exact, run):
    """rms over the channels of (sum - exact result) against the rms of the results; run(shift) -> [.., channels] fp16."""
    shift = (-exact * SCALE).astype(np.float32)
    y = run(shift).astype(np.float64).reshape(-1, exact.size)
    err = (y - (exact * SCALE + shift.astype(np.float64))) / SCALE
    return float(np.sqrt((err ** 2).mean() / (exact ** 2).mean()))


# (channels of all four numbers of steps per unit, reductions of 800 to 25600)
@pytest.mark.parametrize("c,r", [(512, 3), (1024, 3), (128, 5), (1024, 5), (192, 5), (96, 5), (32, 5)])
def test_sums_are_as_exact_as_in_the_kernels_this_one_takes_layers_from(G, c, r):
    """Against the staged kernel, its reduction split over workgroups where the library would."""
    from paper_1904_08368_amd import binding as B
    g = np.random.default_rng(8300 + c + r)
    k = 512
    v, wt = g.standard_normal(c).astype(np.float16), (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
    x = np.ascontiguousarray(np.broadcast_to(v[None, :, None, None], (1, c, r + 2, r + 2)))
    exact = np.einsum("kcrs,c->k", wt.astype(np.float64), v.astype(np.float64))
    d = B.conv_desc(1, c, r + 2, r + 2, k, r, r, 1, 0, B.RELAY_F16, B.RELAY_NHWC, B.HAS_BN)
    assert "igemm_small_kernel" in B.relay_conv2d_kernel_name(d)
    errs = [_sum_errors(exact, lambda sf: G.run_conv_f16(x, wt, 1, 0, scale=np.full(k, SCALE, np.float32), shift=sf, tile=t, split=0).transpose(0, 2, 3, 1))
            for t in (-1, -2)]
    # (an rms over 512 channels of one random filter is known to about 3 %)
    assert errs[0] <= 1.05 * errs[1], errs


@pytest.mark.parametrize("m", [1, 8])
@pytest.mark.parametrize("k", [1024, 4096, 9216, 3168])
def test_dense_sums_are_as_exact_as_lane_by_lane(G, m, k):
    """Against 64 lanes that each add up every 64th group of 8 products in fp32, and their sums in pairs."""
    from paper_1904_08368_amd import binding as B
    g = np.random.default_rng(8400 + k)
    n = 512
    v, w = (g.standard_normal(k) * 128).astype(np.float16), (g.standard_normal((n, k)) * 128 * np.sqrt(2.0 / k)).astype(np.float16)
    prod = w.astype(np.float64) * v.astype(np.float64)
    exact = prod.sum(1) / SCALE

    def run(shift):
        y = torch.full((m, n), float("nan"), dtype=torch.float16, device=G.DEV)
        B.relay_fused_dense_bias_act(m, n, k, B.RELAY_F16, G.up(np.repeat(v[None], m, 0)), G.up(w), G.up(shift), 0, y)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    prod = np.concatenate([prod, np.zeros((n, -k % 512))], axis=1).reshape(n, -1, 64, 8)
    lanes = np.zeros((n, 64), np.float32)
    for i in range(prod.shape[1]):
        for e in range(8):
            lanes = (lanes + prod[:, i, :, e]).astype(np.float32)
    while lanes.shape[1] > 1:
        lanes = lanes[:, : lanes.shape[1] // 2] + lanes[:, lanes.shape[1] // 2:]
    by_lane = float(np.sqrt(((lanes[:, 0] / SCALE - exact) ** 2).mean() / (exact ** 2).mean()))
    err = _sum_errors(exact, run)
    assert err <= 1.05 * by_lane, (err, by_lane)
