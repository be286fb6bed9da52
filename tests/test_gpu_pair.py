"""Two independent convs in one launch: against the oracle, against their own launches, and the errors of the entry point."""
import numpy as np
import pytest
import torch

import oracle as O
from workloads import inputs

# n, c, h, w, k of the two, r of the two, stride; whether they share a launch in fp16 and in int8 (there at least 64 channels).  The staged
# kernel's five tiles (4, 5, 9, 10, 15 of its list), the small-tile kernel, and pairs that stay two launches.
SHAPES = [(1, 128, 28, 28, (256, 256), (3, 1), 2, True, True), (1, 256, 14, 14, (512, 40), (3, 1), 2, True, True),
          (1, 64, 15, 13, (72, 136), (3, 1), 1, False, True), (2, 64, 57, 55, (128, 128), (3, 1), 2, True, True),
          (32, 64, 56, 56, (128, 128), (3, 1), 2, True, True), (16, 128, 28, 28, (256, 256), (3, 1), 2, False, True),
          (1, 32, 5, 3, (8, 24), (1, 3), 1, False, True), (3, 192, 28, 28, (256, 64), (3, 1), 2, True, True),
          (1, 128, 28, 28, (64, 64), (1, 1), 1, True, True), (2, 256, 28, 28, (256, 256), (1, 1), 1, True, True),
          (1, 64, 15, 13, (72, 136), (3, 3), 1, True, True), (1, 128, 14, 14, (128, 64), (3, 3), 1, True, True),
          (2, 96, 9, 11, (40, 40), (1, 1), 1, True, False),
          # 32 x 32 tiles for a pair: 256 of equal reductions, 272 (which is too many), 304 of unequal ones
          (2, 512, 12, 19, (1024, 1024), (1, 1), 2, True, True), (1, 128, 48, 44, (256, 256), (1, 1), 2, True, True),
          (7, 128, 18, 37, (128, 128), (3, 1), 2, True, True)]

def _member(B, G, g, i8, n, c, h, w, k, r, st, relu, res):
    pad = r // 2
    dt = B.RELAY_I8 if i8 else B.RELAY_F16
    if i8:
        wt = g.integers(-127, 128, (k, c, r, r)).astype(np.int8)
        bias = g.integers(-4000, 4000, k).astype(np.int32)
        p = dict(bias=bias, out_rshift=13, relu_flag=relu)
    else:
        wt = (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
        p = dict(scale=(1 + 0.1 * g.standard_normal(k)).astype(np.float32), shift=(0.1 * g.standard_normal(k)).astype(np.float32), relu_flag=relu)
    d = B.conv_desc(n, c, h, w, k, r, r, st, pad, dt, B.RELAY_NHWC, B.flags_of(p.get("bias"), p.get("scale"), None, relu))
    ho, wo = B.relay_conv2d_out_shape(d)
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, G.up(wt), c, wp)
    y = torch.full((n, ho, wo, k), 77, dtype=torch.int8 if i8 else torch.float16, device=G.DEV)
    return d, wt, wp, p, y, dict(stride=(st, st), pad=(pad, pad), **p)


def _oracle_points(g, x, wt, got, oargs, i8):
    """The oracle's values at 200 sampled outputs and the corners, and where they are."""
    pts = [tuple(int(g.integers(e)) for e in got.shape) for _ in range(200)] + [(0, 0, 0, 0), tuple(e - 1 for e in got.shape)]
    acc = O.conv2d_points(x, wt, pts, oargs["stride"], oargs["pad"], integer=i8)
    ks = [t[1] for t in pts]
    if i8:
        return pts, O.requant_points(np.asarray(acc) + oargs["bias"].astype(np.int64)[ks], out_rshift=oargs["out_rshift"], relu_flag=oargs["relu_flag"])
    return pts, O.cast_f16(O.float_epilogue_points(acc, ks, scale=oargs["scale"], shift=oargs["shift"], relu_flag=oargs["relu_flag"]))


@pytest.mark.gpu
@pytest.mark.parametrize("i8", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_pair_matches_oracle_and_separate_launches(shape, i8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    from tests import gpu_util as G
    n, c, h, w, ks, rs, st, *shared = shape
    if i8:
        c = max(c, 64)
    g = np.random.default_rng(inputs.BASE_SEED + 97000 + c + n)
    x = g.integers(-127, 128, (n, c, h, w)).astype(np.int8) if i8 else g.standard_normal((n, c, h, w)).astype(np.float16)
    xd = G.to_nhwc(x, c, B.RELAY_I8 if i8 else B.RELAY_F16)
    calls, refs, ys = [], [], []
    for j in range(2):
        d, wt, wp, p, y, oargs = _member(B, G, g, i8, n, c, h, w, ks[j], rs[j], st, j == 0, None)
        calls.append((d, xd, wp, G.up(p["bias"]), None, 0, p["out_rshift"], y) if i8 else
                     (d, xd, wp, None, G.up(p["scale"]), G.up(p["shift"]), None, y))
        refs.append((wt, oargs))
        ys.append(y)
    assert B.relay_conv2d_pair_fusable(calls[0][0], calls[1][0]) == shared[i8]
    B.relay_conv2d_pair(*calls)
    torch.cuda.synchronize()
    got = [G.from_nhwc(y, k) for y, k in zip(ys, ks)]
    for y in ys:
        y.fill_(55)
    for cl in calls:
        (B.relay_qconv2d_requant if i8 else B.relay_fused_conv2d_bias_bn_relu)(*cl)
    torch.cuda.synchronize()
    for a, y, k, (wt, oargs) in zip(got, ys, ks, refs):
        assert np.array_equal(a.view(np.uint8), G.from_nhwc(y, k).view(np.uint8))
        pts, want = _oracle_points(g, x, wt, a, oargs, i8)
        at = np.array([a[t] for t in pts])
        if i8:
            assert np.array_equal(at, want)
        else:   # (one fp16 unit in the last place, or 1e-5 of the result's scale in the fp32 sums)
            rms = float(np.sqrt(np.mean(a.astype(np.float64) ** 2)))
            err = np.abs(at.astype(np.float64) - want.astype(np.float64)) / np.maximum(np.abs(want.astype(np.float64)), rms)
            assert err.max() <= 2.0 ** -10 + 1e-5


def test_pair_checks_and_rule_on_the_host():
    import ctypes as C
    from paper_1904_08368_amd import binding as B
    d = lambda n, c, hw, k, r, st=2, dt=B.RELAY_F16: B.conv_desc(n, c, hw, hw, k, r, r, st, r // 2, dt, B.RELAY_NHWC, 0)
    assert B.relay_conv2d_pair_fusable(d(1, 128, 28, 256, 3), d(1, 128, 28, 256, 1))          # 32 staged 64 x 64 tiles
    assert not B.relay_conv2d_pair_fusable(d(1, 128, 28, 256, 3, 1), d(1, 128, 28, 256, 1, 1))  # fp16: small tiles would sum the second differently
    assert B.relay_conv2d_pair_fusable(d(1, 128, 28, 256, 3, dt=B.RELAY_I8), d(1, 128, 28, 256, 1, dt=B.RELAY_I8))  # small tiles, two to a CU
    assert not B.relay_conv2d_pair_fusable(d(16, 256, 14, 512, 3, dt=B.RELAY_I8), d(16, 256, 14, 512, 1, dt=B.RELAY_I8))  # one to a CU: two rounds
    assert B.relay_conv2d_pair_fusable(d(32, 64, 56, 128, 3), d(32, 64, 56, 128, 1))          # the staged kernel's 128 x 64 tile
    assert not B.relay_conv2d_pair_fusable(d(32, 128, 28, 128, 3, 1), d(32, 128, 28, 128, 1, 1))   # the 3x3 kernel runs the first
    with pytest.raises(B.RelayError) as e:
        B.relay_conv2d_pair_fusable(d(1, 64, 8, 64, 3), d(1, 64, 8, 64, 1, dt=B.RELAY_I8))
    assert e.value.status == 3
    F = 1 << 30
    dd = d(1, 64, 8, 64, 3)
    call = lambda y, x=F, res=None, **kw: B.ConvCall(*{**dict(d=C.pointer(dd), x=x, w=F + 4096, b=None, sc=None, sf=None, res=res, l=0, r=0, y=y), **kw}.values())
    run = lambda a, b: B.lib().relay_conv2d_pair(C.byref(a), C.byref(b), None)
    assert run(call(F + 8192), call(F + 8192)) == 4                   # one output
    assert run(call(F + 8192), call(F + 16384, x=F + 8192)) == 4      # the second reads the first's output
    assert run(call(F + 8192, res=F + 16384), call(F + 16384)) == 4
    for kw in (dict(w=F + 8192), dict(b=F + 8192), dict(sc=F + 8192), dict(sf=F + 8192)):     # filters and constants, either way round
        assert run(call(F + 8192), call(F + 16384, **kw)) == 4
        assert b"one conv's output" in B.lib().relay_last_error()
        assert run(call(F + 16384, **kw), call(F + 8192)) == 4
        assert b"one conv's output" in B.lib().relay_last_error()
    assert run(call(F + 8200), call(F + 16384)) == 5                  # a member's own checks
    assert run(call(None), call(F + 16384)) == 1
    assert B.lib().relay_conv2d_pair(None, C.byref(call(F)), None) == 1
