"""GPU parity of the dense kernels and the two layout-side kernels at the edges of their rules: few and many rows, units
that are no multiple of 8, reductions on both sides of the split; pixel counts around a vector and channel counts
around a block; average pools of fewer and more positions than a workgroup has threads for."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu
# Both sides round to fp16: one unit in the last place where the fp32 sums fall on the other side of a boundary.
TOL_F16 = 2.0 ** -10 + 1e-5


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("m,n,k", [(1, 1000, 512), (1, 18, 512), (4, 10, 2048), (5, 10, 2048), (1, 7, 3136), (15, 33, 96),
                                   (16, 64, 64), (17, 1000, 1024), (3, 40, 72), (70, 24, 32)])
@pytest.mark.parametrize("act", [0, 1])
def test_dense_matches_the_oracle(G, m, n, k, act):
    from paper_1904_08368_amd import binding as B
    g = np.random.default_rng(9100 + m + n + k)
    x = g.standard_normal((m, k)).astype(np.float16)
    w = (g.standard_normal((n, k)) / np.sqrt(k)).astype(np.float16)
    b = g.standard_normal(n).astype(np.float32)
    y = torch.full((m, n), float("nan"), dtype=torch.float16, device=G.DEV)
    B.relay_fused_dense_bias_act(m, n, k, B.RELAY_F16, G.up(x), G.up(w), G.up(b), act, y)
    torch.cuda.synchronize()
    want = O.fused_dense(x, w, bias=b, relu_flag=bool(act), out_dtype="f16")
    assert O.max_rel_err(y.cpu().numpy(), want) <= TOL_F16


# one row or more, units and reductions on both sides of the rule that gives a workgroup to an output unit; reductions the
# small-tile kernel does not take
@pytest.mark.parametrize("m,n,k", [(2, 1024, 2048), (2, 1032, 2048), (3, 24, 2048), (3, 24, 8192), (4, 40, 2056), (4, 2056, 2056), (1, 20, 40),
                                   (9, 20, 40), (33, 12, 72)])
def test_dense_on_both_sides_of_its_rules(G, m, n, k):
    test_dense_matches_the_oracle(G, m, n, k, 1)


@pytest.mark.parametrize("m,n,k", [(1, 9, 36), (1, 30, 1028), (2, 9, 36), (8, 5, 260), (9, 30, 1028), (33, 12, 516)])
def test_dense_fp32_matches_the_oracle(G, m, n, k):
    from paper_1904_08368_amd import binding as B
    g = np.random.default_rng(9150 + m + n + k)
    x, w = g.standard_normal((m, k)).astype(np.float32), (g.standard_normal((n, k)) / np.sqrt(k)).astype(np.float32)
    b = g.standard_normal(n).astype(np.float32)
    y = torch.full((m, n), float("nan"), dtype=torch.float32, device=G.DEV)
    B.relay_fused_dense_bias_act(m, n, k, B.RELAY_F32, G.up(x), G.up(w), G.up(b), 1, y)
    torch.cuda.synchronize()
    want = np.maximum(x.astype(np.float64) @ w.astype(np.float64).T + b, 0)
    # at most 20 rounded sums in a row per lane, 6 across the lanes: under 26 half-units of the largest partial sum (below 4)
    assert np.abs(y.cpu().numpy() - want).max() <= 26 * 2.0 ** -24 * 4


def test_dense_takes_outputs_of_element_alignment(G):
    from paper_1904_08368_amd import binding as B
    g = np.random.default_rng(9200)
    x, w = g.standard_normal((3, 64)).astype(np.float16), (g.standard_normal((16, 64)) / 8).astype(np.float16)
    buf = torch.full((3 * 16 + 1,), float("nan"), dtype=torch.float16, device=G.DEV)
    B.relay_fused_dense_bias_act(3, 16, 64, B.RELAY_F16, G.up(x), G.up(w), None, 0, buf[1:])
    torch.cuda.synchronize()
    want = O.fused_dense(x, w, bias=None, relu_flag=False, out_dtype="f16")
    assert O.max_rel_err(buf[1:].cpu().numpy().reshape(3, 16), want) <= TOL_F16


@pytest.mark.parametrize("dtype", [np.float16, np.int8])
@pytest.mark.parametrize("n,c,h,w,pad", [(1, 1, 1, 1, 15), (2, 3, 1, 7, 5), (2, 5, 2, 4, 11), (3, 37, 3, 3, 43), (1, 64, 5, 13, 0),
                                         (2, 70, 8, 8, 10), (1, 129, 7, 11, 31), (2, 16, 1, 3, 0), (1, 9, 6, 5, 4)])
def test_layout_conversion_at_vector_edges(G, dtype, n, c, h, w, pad):
    """(the last shape has a padded channel count that takes the element-wise kernel)"""
    from paper_1904_08368_amd import binding as B
    x = np.random.default_rng(9300 + c).integers(-127, 128, (n, c, h, w)).astype(dtype)
    cp = c + pad
    y = torch.full((n, h, w, cp), 7, dtype=torch.float16 if dtype is np.float16 else torch.int8, device=G.DEV)
    B.relay_nchw_to_nhwc(B.RELAY_F16 if dtype is np.float16 else B.RELAY_I8, n, c, h, w, cp, G.up(x), y)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.array_equal(got[..., :c], x.transpose(0, 2, 3, 1)) and not got[..., c:].any()


@pytest.mark.parametrize("n,c,h,w,pad", [(3, 37, 47, 43, 11), (40, 129, 7, 11, 31), (1600, 16, 2, 4, 0), (1, 1, 113, 117, 15), (2100, 70, 1, 5, 10)])
def test_int8_layout_conversion_in_pieces(G, n, c, h, w, pad):
    """The sizes from which int8 takes whole vectors, with ragged pixel counts, channels and channel blocks."""
    test_layout_conversion_at_vector_edges(G, np.int8, n, c, h, w, pad)


@pytest.mark.parametrize("n,c,hw", [(1, 8, 1), (2, 24, 31), (1, 72, 33), (3, 512, 49), (1, 64, 500)])
def test_average_pool_matches_the_mean(G, n, c, hw):
    from paper_1904_08368_amd import binding as B
    x = np.random.default_rng(9400 + c).standard_normal((n, hw, c)).astype(np.float16)
    y = torch.full((n, c), float("nan"), dtype=torch.float16, device=G.DEV)
    B.relay_global_avgpool(B.RELAY_F16, n, c, hw, G.up(x), y)
    torch.cuda.synchronize()
    want = x.astype(np.float64).mean(axis=1).astype(np.float16)
    assert O.max_rel_err(y.cpu().numpy(), want) <= TOL_F16


@pytest.mark.parametrize("n,c,hw", [(2, 520, 3), (1, 264, 9), (2, 136, 25), (3, 64, 32), (2, 24, 100), (1, 16, 200), (3, 8, 300), (2, 8, 5)])
def test_average_pool_with_every_number_of_channel_vectors(G, n, c, hw):
    """64, 32, 16, 8, 4, 2 and 1 channel vectors a workgroup, and fewer vectors than that."""
    test_average_pool_matches_the_mean(G, n, c, hw)


@pytest.mark.parametrize("dtype", [np.float16, np.int8])
@pytest.mark.parametrize("n,c,h,w,r", [(1, 3, 5, 7, 7), (2, 4, 9, 16, 3), (3, 1, 1, 9, 1), (2, 2, 13, 2, 3), (4, 3, 226, 221, 7), (5, 4, 200, 202, 5)])
def test_padded_copy_of_the_image(G, dtype, n, c, h, w, r):
    """One and (fp16, the last two) two pixels per thread; every side of the image on and off a whole group of pixels."""
    from paper_1904_08368_amd import binding as B
    p = r // 2
    dt = B.RELAY_F16 if dtype is np.float16 else B.RELAY_I8
    x = np.random.default_rng(9500 + h).integers(-127, 128, (n, c, h, w)).astype(dtype)
    d = B.conv_desc(n, c, h, w, 8, r, r, 1, p, dt, B.RELAY_NHWC4_PADDED, 0)
    hp, wp = B.relay_nhwc4_padded_shape(d)
    y = torch.full((n, hp, wp, 4), 7, dtype=torch.float16 if dtype is np.float16 else torch.int8, device=G.DEV)
    B.relay_pack_input_nhwc4(d, G.up(x), y)
    torch.cuda.synchronize()
    want = np.zeros((n, hp, wp, 4), dtype)
    want[:, p:p + h, p:p + w, :c] = x.transpose(0, 2, 3, 1)
    assert np.array_equal(y.cpu().numpy(), want)
