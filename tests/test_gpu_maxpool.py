"""The 3x3 max pools (one and two outputs per thread) and the padded NHWC4 copy against plain numpy, element for element:
ragged sizes, one-pixel images, the lowest values, infinities, and NaN as a first and as a later tap (the rule is "larger than the
best so far": a NaN counts only where the window begins with it)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _pool(x, r, st, pd):
    """x [n, h, w, c]; taps in row order, those outside the image left out."""
    n, h, w, c = x.shape
    ho, wo = (h + 2 * pd - r) // st + 1, (w + 2 * pd - r) // st + 1
    best, have = np.zeros((n, ho, wo, c), dtype=x.dtype), np.zeros((1, ho, wo, 1), dtype=bool)
    for a in range(r):
        for b in range(r):
            ih, iw = np.arange(ho) * st - pd + a, np.arange(wo) * st - pd + b
            ok = (((ih >= 0) & (ih < h))[:, None] & ((iw >= 0) & (iw < w))[None, :])[None, :, :, None]
            v = x[:, np.clip(ih, 0, h - 1)][:, :, np.clip(iw, 0, w - 1)]
            with np.errstate(invalid="ignore"):
                best = np.where(ok & (~have | (v > best)), v, best)
            have = have | ok
    return best


@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("shape", [(2, 1, 1, 16, 1, 1), (3, 5, 1, 32, 1, 1), (2, 7, 9, 48, 1, 1), (2, 9, 7, 32, 2, 1), (2, 9, 8, 16, 2, 0),
                                   (11, 29, 27, 512, 1, 1), (22, 29, 27, 512, 1, 0), (1, 28, 28, 256, 3, 1)])
def test_maxpool3(shape, i8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    n, h, w, c, st, pd = shape
    g = np.random.default_rng(h * w + c + st)
    if i8:
        x = g.integers(-128, 128, (n, h, w, c)).astype(np.int8)
        x[0] = -128
    else:
        x = g.standard_normal((n, h, w, c)).astype(np.float16)
        x[0] = -65504
        x[-1, ..., 3] = -np.inf
        x[-1, ..., 4] = np.inf
        x[g.random(x.shape) < 0.05] = np.nan
        x[..., 5] = np.nan
    want = _pool(x, 3, st, pd)
    y = torch.empty(want.shape, dtype=torch.int8 if i8 else torch.float16, device="cuda:0")
    B.relay_maxpool2d(B.RELAY_I8 if i8 else B.RELAY_F16, n, c, h, w, 3, st, pd, torch.from_numpy(x).cuda(), y)
    assert np.array_equal(y.cpu().numpy(), want, equal_nan=not i8)


@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 3, 1), (2, 3, 5, 7, 3, 1), (1, 4, 84, 84, 8, 0), (3, 2, 17, 31, 7, 3), (2, 3, 64, 250, 3, 1)])
def test_padded_nhwc4(shape, i8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    n, c, h, w, r, pd = shape
    g = np.random.default_rng(h * w + c)
    x = g.integers(-128, 128, (n, c, h, w)).astype(np.int8 if i8 else np.float16)
    d = B.conv_desc(n, c, h, w, 8, r, r, 1, pd, B.RELAY_I8 if i8 else B.RELAY_F16, B.RELAY_NHWC4_PADDED, 0)
    hp, wp = B.relay_nhwc4_padded_shape(d)
    want = np.zeros((n, hp, wp, 4), dtype=x.dtype)
    want[:, pd:pd + h, pd:pd + w, :c] = x.transpose(0, 2, 3, 1)
    y = torch.full(want.shape, 9, dtype=torch.int8 if i8 else torch.float16, device="cuda:0")
    B.relay_pack_input_nhwc4(d, torch.from_numpy(x).cuda(), y)
    assert np.array_equal(y.cpu().numpy(), want)
