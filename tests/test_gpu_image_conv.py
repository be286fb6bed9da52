"""The first-layer conv on the NCHW image, with and without the max pool behind it, against the separate calls: the padded copy,
the conv over it, the pool."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as O
from workloads import inputs

# n, c, h, w, k, window, stride, pad, pooled: large and small tiles, 64 and 32 channels and ragged ones, images that end inside a tile, odd
# widths (single pixels) and even ones (pairs), one and two k-steps per filter row, a pooled map whose last windows stick out
SHAPES = [(1, 3, 224, 224, 64, 7, 2, 3, True), (2, 3, 61, 45, 64, 7, 2, 3, True), (3, 3, 33, 70, 80, 7, 2, 3, True), (24, 3, 57, 64, 64, 7, 2, 3, True),
          (1, 4, 84, 84, 32, 8, 4, 0, False), (40, 4, 84, 84, 32, 8, 4, 0, False), (1, 3, 17, 15, 64, 3, 1, 1, False), (3, 3, 130, 97, 64, 3, 1, 1, False),
          (2, 3, 163, 206, 32, 3, 2, 1, False), (30, 3, 64, 50, 32, 3, 2, 1, False), (1, 1, 5, 4, 8, 5, 2, 2, False), (2, 2, 1, 2, 48, 7, 2, 3, True)]


def _calls(G, B, i8, x, wt, p, d, ho, wo, pooled):
    """The separate calls' conv output and pooled output (NHWC, on the device) and the operands."""
    n, c, k = x.shape[0], x.shape[1], wt.shape[0]
    dt, tdt = (B.RELAY_I8, torch.int8) if i8 else (B.RELAY_F16, torch.float16)
    hp, wp = B.relay_nhwc4_padded_shape(d)
    xd, packed = G.up(x), torch.empty((n, hp, wp, 4), dtype=tdt, device=G.DEV)
    w = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, G.up(wt), c, w)
    y = torch.zeros((n, ho, wo, k), dtype=tdt, device=G.DEV)
    yp = torch.zeros((n, (ho - 1) // 2 + 1, (wo - 1) // 2 + 1, k), dtype=tdt, device=G.DEV)
    B.relay_pack_input_nhwc4(d, xd, packed)
    if i8:
        B.relay_qconv2d_requant(d, packed, w, p["b"], None, 0, p["s"], y, None)
    else:
        B.relay_fused_conv2d_bias_bn_relu(d, packed, w, p["b"], p["sc"], p["sf"], None, y, None)
    if pooled:
        B.relay_maxpool2d(dt, n, k, ho, wo, 3, 2, 1, y, yp)
    return xd, w, y, yp


@pytest.mark.gpu
@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_image_conv_gives_the_results_of_the_separate_calls(shape, i8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    from tests import gpu_util as G
    n, c, h, w, k, r, st, pad, pooled = shape
    g = np.random.default_rng(inputs.BASE_SEED + 99000 + h + k)
    if i8:
        x, wt = (g.integers(-127, 128, e).astype(np.int8) for e in ((n, c, h, w), (k, c, r, r)))
        p = dict(b=G.up(g.integers(-4000, 4000, k).astype(np.int32)), s=9)
        flags = B.HAS_BIAS | B.RELU
    else:
        x = g.standard_normal((n, c, h, w)).astype(np.float16)
        wt = (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
        p = {a: G.up((m + 0.1 * g.standard_normal(k)).astype(np.float32)) for a, m in (("b", 0), ("sc", 1), ("sf", 0))}
        flags = B.HAS_BIAS | B.HAS_BN | B.RELU
    d = B.conv_desc(n, c, h, w, k, r, r, st, pad, B.RELAY_I8 if i8 else B.RELAY_F16, B.RELAY_NHWC4_PADDED, flags)
    assert B.relay_image_conv2d_supported(d, pooled) == (not i8 or st % 2 == 0)
    if i8 and st % 2:
        return
    ho, wo = B.relay_conv2d_out_shape(d)
    xd, wp, y0, yp0 = _calls(G, B, i8, x, wt, p, d, ho, wo, pooled)
    for conv_too in ((True, False) if pooled else (True,)):
        y, yp = torch.full_like(y0, 77), torch.full_like(yp0, 77)
        outs = (y if conv_too else None, yp if pooled else None)
        if i8:
            B.relay_qimage_conv2d(d, xd, wp, p["b"], p["s"], *outs)
        else:
            B.relay_fused_image_conv2d(d, xd, wp, p["b"], p["sc"], p["sf"], *outs)
        torch.cuda.synchronize()
        for got, want, used in ((y, y0, conv_too), (yp, yp0, pooled)):
            if not used:
                assert bool((got == 77).all())
            elif i8:
                assert torch.equal(got, want)
            else:   # the same fp32 sums up to their grouping (1e-6 of the outputs' size): a rounding to fp16 may go the other way, one ulp
                assert O.max_rel_err(got.cpu().numpy(), want.cpu().numpy()) <= 1.1 * 2.0 ** -10


def test_image_conv_argument_checks():
    from paper_1904_08368_amd import binding as B
    ok = dict(dtype=B.RELAY_F16, layout=B.RELAY_NHWC4_PADDED, flags=B.RELU)

    def desc(n=1, c=3, h=32, w=32, k=64, r=7, st=2, pad=3, **kw):
        e = dict(ok, **kw)
        return B.conv_desc(n, c, h, w, k, r, r, st, pad, e["dtype"], e["layout"], e["flags"])
    assert B.relay_image_conv2d_supported(desc(), True) and B.relay_image_conv2d_supported(desc(), False)
    for bad in (desc(layout=B.RELAY_NHWC), desc(flags=B.RELU | B.HAS_RESIDUAL), desc(k=60), desc(r=11, pad=5), desc(dtype=B.RELAY_I8, st=1),
                desc(dtype=B.RELAY_I8, flags=B.HAS_BN), desc(c=5)):
        assert not B.relay_image_conv2d_supported(bad, False)
    assert not B.relay_image_conv2d_supported(desc(flags=0), True)      # a float pool without relu

    # taken, and slower than the separate calls: large patches read for several channel tiles, or pixel by pixel
    dqn = dict(c=4, h=84, w=84, k=32, r=8, st=4, pad=0)
    for d, pooled, pays in ((desc(), True, True), (desc(**dqn), False, True), (desc(**dict(dqn, w=83)), False, False),
                            (desc(n=20, h=198, w=31, k=128, r=3, st=4, pad=1), False, False), (desc(n=40, h=71, w=202, k=128, r=8, st=4, pad=3), True, False),
                            (desc(n=40, h=71, w=202, k=64, r=8, st=4, pad=3), True, True), (desc(k=60), False, False)):
        assert B.relay_image_conv2d_pays(d, pooled) == pays
    # more workgroups than one launch holds; the most of which the smaller ones still fit
    assert not B.relay_image_conv2d_supported(desc(n=20000000, c=1, h=1, w=2, k=64, r=1, st=1, pad=0), False)
    assert B.relay_image_conv2d_supported(desc(n=16000000, c=1, h=1, w=2, k=64, r=1, st=1, pad=0), False)
    assert B.relay_image_conv2d_supported(desc(n=20000000, c=1, h=1, w=2, k=8, r=1, st=1, pad=0), False)
    assert not B.relay_image_conv2d_supported(desc(c=1, h=1, w=2, k=5000000, r=1, st=1, pad=0), False)

    x, w, y = 0x7F0000000000, 0x7F0000100000, 0x7F0000200000     # (never dereferenced: every call is refused)
    for args, status in (((None, w, y, None), 1), ((x, w, None, None), 1), ((x, w, x, None), 4), ((x, w, y, y), 4), ((x + 2, w, y, None), 5),
                         ((x, w + 8, y, None), 5), ((x, w, y + 8, None), 5)):
        got = B.lib().relay_fused_image_conv2d(C.byref(desc()), args[0], args[1], None, None, None, args[2], args[3], None)
        assert got == status, (status, got, B.lib().relay_last_error())


# infinities and a NaN in some pixels of the first image: they reach the outputs whose window they lie in, and those whose filter row,
# filled up with zeros to 4 or 8 columns, ends on them; all others are what they would be
@pytest.mark.gpu
@pytest.mark.parametrize("finite", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_image_conv_against_64_bits(shape, finite):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import torch.nn.functional as F
    from paper_1904_08368_amd import binding as B
    from tests import gpu_util as G
    n, c, h, w, k, r, st, pad, pooled = shape
    g = np.random.default_rng(inputs.BASE_SEED + 99500 + h + k)
    x = torch.from_numpy(g.standard_normal((n, c, h, w)).astype(np.float16))
    wt = torch.from_numpy((g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16))
    b, sc, sf = (torch.from_numpy((m + 0.1 * g.standard_normal(k)).astype(np.float32)) for m in (0, 1, 0))
    bad = torch.zeros((n, 1, h, w))
    xb = x.clone()
    if not finite:
        for v in (np.inf, -np.inf, np.nan):
            i, j = int(g.integers(h)), int(g.integers(w))
            xb[0, int(g.integers(c)), i, j] = v
            bad[0, 0, i, j] = 1
    d = B.conv_desc(n, c, h, w, k, r, r, st, pad, B.RELAY_F16, B.RELAY_NHWC4_PADDED, B.HAS_BIAS | B.HAS_BN | B.RELU)
    ho, wo = B.relay_conv2d_out_shape(d)
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, wt.to(G.DEV), c, wp)
    y = torch.full((n, ho, wo, k), -7.0, dtype=torch.float16, device=G.DEV)
    yp = torch.full((n, (ho - 1) // 2 + 1, (wo - 1) // 2 + 1, k), -7.0, dtype=torch.float16, device=G.DEV)
    B.relay_fused_image_conv2d(d, xb.to(G.DEV), wp, b.to(G.DEV), sc.to(G.DEV), sf.to(G.DEV), y, yp if pooled else None)
    torch.cuda.synchronize()
    col = lambda v: v.double().reshape(1, k, 1, 1)
    conv = lambda a, f: F.conv2d(a.double(), f.double(), stride=st, padding=pad)
    ref = (conv(x, wt) + col(b)) * col(sc) + col(sf)
    # half a unit of the fp16 result, and the fp32 sums: at most c r r + 4 roundings of partial sums below that of the magnitudes
    tol = 2.0 ** -11 * ref.abs() + 2.0 ** -24 + (c * r * r + 4) * 2.0 ** -24 * ((conv(x.abs(), wt.abs()) + col(b).abs()) * col(sc).abs() + col(sf).abs())
    cols = 4 if r <= 4 else 8
    reach = F.conv2d(F.pad(bad, (pad, pad + cols - r, pad, pad)), torch.ones(1, 1, r, cols), stride=st)[..., :wo] > 0
    assert finite or int(reach.sum()) < reach.numel() or h * w < 30
    got = y.cpu().double().permute(0, 3, 1, 2)
    off = ((got - ref.clamp(min=0)).abs() <= tol) | reach
    assert bool(off.all())
    if pooled:
        pool = lambda a: F.max_pool2d(a, 3, 2, 1)
        got = yp.cpu().double().permute(0, 3, 1, 2)
        lo, hi = pool((ref - tol).clamp(min=0)), pool((ref + tol).clamp(min=0))
        assert bool((((got >= lo) & (got <= hi)) | (pool(reach.double()) > 0)).all())


# deep Q-network, ResNet's and VGG's first layers at sizes where the conv over the padded copy splits its sums over four waves (and
# one where it does not): the fp32 sums against 64 bits, seen through a scale and shift that leave little but their error
@pytest.mark.gpu
@pytest.mark.parametrize("n,c,h,w,k,r,st,pad,pooled", [(11, 4, 84, 84, 32, 8, 4, 0, False), (32, 4, 84, 84, 32, 8, 4, 0, False), (8, 3, 64, 64, 64, 7, 2, 3, True),
                                                       (2, 3, 128, 128, 64, 7, 2, 3, True), (1, 3, 64, 64, 64, 3, 1, 1, False), (2, 3, 224, 224, 64, 7, 2, 3, True)])
def test_sums_are_no_less_exact_than_those_of_the_separate_calls(n, c, h, w, k, r, st, pad, pooled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    from tests import gpu_util as G
    d = B.conv_desc(n, c, h, w, k, r, r, st, pad, B.RELAY_F16, B.RELAY_NHWC4_PADDED, B.HAS_BN | B.RELU)
    ho, wo = B.relay_conv2d_out_shape(d)
    oy, ox = ho // 2, wo // 2
    errors = ([], [])
    for seed in range(40):
        g = np.random.default_rng(seed)
        x = np.repeat(g.standard_normal((1, c, h, w)).astype(np.float16), n, axis=0)
        wt = (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
        y0, x0 = oy * st - pad, ox * st - pad
        e = 2.0 ** 20 * np.einsum("kcrs,crs->k", wt.astype(np.float64), x[0, :, y0:y0 + r, x0:x0 + r].astype(np.float64))
        # 2^20 acc + 8 - round(e): a whole number below 2^24 is taken from a sum beside it, exact in fp32, and 2^-7 is fp16's step at 8
        p = dict(b=None, sc=torch.full((k,), 2.0 ** 20, device=G.DEV), sf=G.up((8.0 - np.round(e)).astype(np.float32)))
        xd, wp, y, yp = _calls(G, B, False, x, wt, p, d, ho, wo, pooled)
        z, zp = torch.empty_like(y), torch.empty_like(yp)
        B.relay_fused_image_conv2d(d, xd, wp, None, p["sc"], p["sf"], z, zp if pooled else None)
        torch.cuda.synchronize()
        for out, t in zip(errors, (y, z)):
            out.append(t[n - 1, oy, ox].double().cpu().numpy() - 8.0 + np.round(e) - e)
    two, one = (np.sqrt(np.mean(np.concatenate(v) ** 2)) * 2.0 ** -20 for v in errors)
    print(f"[observed] rms of the sums' errors, {n} x {h} x {w}, {r} x {r}: separate calls {two:.2e}, one launch {one:.2e}")
    # (the same sums in as many runs: only how a matrix instruction adds up its 16 or 32 products differs; half the runs are 1.08 to 1.5 times)
    assert one <= 1.03 * two


# Small tiles with helper waves (at most 512 workgroups) and without, at 32 and at 64 channels, pixel pairs and single pixels: a patch of
# more pixels than threads and of fewer, channels past the tile's, workgroups of more than one channel tile.
@pytest.mark.gpu
@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("shape", [(1, 4, 84, 84, 32, 8, 4, 0, False), (2, 4, 61, 85, 24, 8, 4, 3, False), (1, 3, 9, 8, 8, 3, 1, 1, False),
                                   (1, 3, 61, 62, 64, 5, 2, 2, False), (1, 4, 40, 71, 72, 8, 4, 0, False),
                                   (129, 4, 84, 84, 32, 8, 5, 0, False), (65, 4, 84, 84, 96, 8, 6, 4, False)])
def test_small_tiles_with_and_without_helper_waves(shape, i8):
    test_image_conv_gives_the_results_of_the_separate_calls(shape, i8)
