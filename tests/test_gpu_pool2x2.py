"""3x3 conv with the 2x2 max pool behind it as one launch: both results bit for bit those of the two launches."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    from tests import gpu_util
    return gpu_util


# 16 x 16 tiles: whole, cut on both sides, a single window, several images; a chunk of 64 channels, several of 32; filters that
# end inside a tile
@pytest.mark.parametrize("bias,bn", [(True, False), (False, True)])
@pytest.mark.parametrize("shape", [(2, 64, 16, 32, 64), (1, 96, 18, 30, 72), (3, 128, 2, 2, 40), (1, 64, 34, 14, 136)])
def test_equals_conv_then_pool(G, shape, bias, bn):
    from paper_1904_08368_amd import binding as B
    n, c, h, w, k = shape
    g = torch.Generator(device=G.DEV)
    g.manual_seed(h * w + k)
    rnd = lambda *s: torch.randn(s, device=G.DEV, generator=g)
    x, wt = rnd(n, h, w, c).half(), (rnd(k, c, 3, 3) * (2.0 / (9 * c)) ** 0.5).half()
    b, sc, sf = (rnd(k) if bias else None), (rnd(k) if bn else None), (rnd(k) if bn else None)
    d = B.conv_desc(n, c, h, w, k, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(b, sc, None, True))
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, wt, c, wp)
    y, yp = (torch.full((n, h // s, w // s, k), -7.0, dtype=torch.float16, device=G.DEV) for s in (1, 2))
    z, zp = torch.empty_like(y), torch.empty_like(yp)
    B.relay_set_conv_tile(105)      # the 16 x 16 tiles
    try:
        assert B.relay_conv2d_pool2x2_pays(d)
        B.relay_fused_conv2d_bias_bn_relu(d, x, wp, b, sc, sf, None, z, None)
    finally:
        B.relay_set_conv_tile(-1)
    B.relay_maxpool2d(B.RELAY_F16, n, k, h, w, 2, 2, 0, z, zp)
    B.relay_fused_conv2d_pool2x2(d, x, wp, b, sc, sf, y, yp)
    torch.cuda.synchronize()
    assert torch.equal(y, z) and torch.equal(yp, zp)


def test_a_forced_tile_gets_the_two_launches(G):
    """128 channels, which the 16 x 16 tiles add up in another order than the implicit GEMM that is asked for."""
    from paper_1904_08368_amd import binding as B
    n, c, h, w, k = 3, 128, 34, 30, 72
    g = torch.Generator(device=G.DEV)
    g.manual_seed(7)
    x, wt = torch.randn((n, h, w, c), device=G.DEV, generator=g).half(), (torch.randn((k, c, 3, 3), device=G.DEV, generator=g) * 0.04).half()
    d = B.conv_desc(n, c, h, w, k, 3, 3, 1, 1, B.RELAY_F16, B.RELAY_NHWC, B.RELU)
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=G.DEV)
    B.relay_prepack_conv2d_weights(d, wt, c, wp)
    outs = {}
    for tile in (-2, 105):
        y, yp = (torch.full((n, h // s, w // s, k), -7.0, dtype=torch.float16, device=G.DEV) for s in (1, 2))
        z, zp = torch.empty_like(y), torch.empty_like(yp)
        B.relay_set_conv_tile(tile)
        try:
            B.relay_fused_conv2d_pool2x2(d, x, wp, None, None, None, y, yp)
            B.relay_fused_conv2d_bias_bn_relu(d, x, wp, None, None, None, None, z, None)
        finally:
            B.relay_set_conv_tile(-1)
        B.relay_maxpool2d(B.RELAY_F16, n, k, h, w, 2, 2, 0, z, zp)
        torch.cuda.synchronize()
        assert torch.equal(y, z) and torch.equal(yp, zp)
        outs[tile] = y
    assert not torch.equal(outs[-2], outs[105])


def test_what_is_refused(G):
    from paper_1904_08368_amd import binding as B
    t = torch.zeros(1 << 16, dtype=torch.float16, device=G.DEV)
    desc = lambda **o: B.conv_desc(**{**dict(n=1, c=64, h=8, w=8, k=64, r=3, s=3, stride=1, pad=1, dtype=B.RELAY_F16, layout=B.RELAY_NHWC,
                                             flags=B.RELU), **o})
    for d in (desc(flags=0), desc(h=7), desc(w=9), desc(k=60), desc(stride=2), desc(r=1, s=1, pad=0), desc(dtype=B.RELAY_I8)):
        assert not B.relay_conv2d_pool2x2_pays(d)
        with pytest.raises(B.RelayError):
            B.relay_fused_conv2d_pool2x2(d, t, t[8192:], None, None, None, t[16384:], t[32768:])
    with pytest.raises(B.RelayError):
        B.relay_fused_conv2d_pool2x2(desc(), t, t[8192:], None, None, None, t[16384:], t[16384:])


def test_networks_use_it_and_keep_both_tensors(G):
    """Four 3x3 convs and two 2x2 pools, plain calls against the merged ones."""
    import numpy as np
    from paper_1904_08368_amd.fusion import FusedOp
    from paper_1904_08368_amd.stack import FusedNet
    ops, cur, cin = [], "x", 64
    for i, k in enumerate((64, 128)):
        ops.append(FusedOp("conv", f"c{i}", cur, f"t{i}", cin, k, 3, 1, 1, bias=True, relu=True))
        ops.append(FusedOp("maxpool", f"p{i}", f"t{i}", f"u{i}", k, k, 2, 2, 0))
        cur, cin = f"u{i}", k
    rng = np.random.default_rng(5)
    params = [dict(w=(rng.standard_normal((o.cout, o.cin, 3, 3)) * 0.06).astype(np.float16), bias=rng.standard_normal(o.cout).astype(np.float32))
              if o.kind == "conv" else {} for o in ops]
    net = FusedNet(ops, params, 8, 128, 128, "f16", in_channels=64)
    net.load_input(rng.standard_normal((8, 64, 128, 128)).astype(np.float16))
    assert net.merged
    got = []
    for merged in (net.merged, {}):
        net.merged = merged
        net.run()
        torch.cuda.synchronize()
        got.append({k: net.bufs[k].clone() for k in ("t0", "u0", "t1", "u1")})
        for k in ("t0", "u0", "t1", "u1"):
            net.bufs[k].zero_()
    assert all(torch.equal(got[0][k], got[1][k]) for k in got[0])
