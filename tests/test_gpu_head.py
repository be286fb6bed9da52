"""Global average pool + dense as one launch, against the same fp16 roundings in 64-bit arithmetic."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    from tests import gpu_util
    return gpu_util


# units that fill no workgroup, channels at and beside the
# sizes where a thread's share changes, one position, more positions than a round takes
@pytest.mark.parametrize("n,c,hw,units", [(1, 512, 49, 1000), (1, 8, 1, 1), (1, 520, 7, 9), (3, 1024, 56, 1000), (5, 2048, 4, 2100),
                                          (9, 72, 49, 1000), (11, 1024, 42, 1000), (13, 1032, 100, 999), (32, 512, 49, 1000),
                                          (33, 24, 300, 1000), (70, 64, 64, 33)])
@pytest.mark.parametrize("act", [0, 1])
def test_pool_and_dense(G, n, c, hw, units, act):
    from paper_1904_08368_amd import binding as B
    g = torch.Generator(device=G.DEV)
    g.manual_seed(n * c + hw)
    x = torch.randn((n, hw, c), device=G.DEV, generator=g).half()
    w = (torch.randn((units, c), device=G.DEV, generator=g) / c ** 0.5).half()
    b = torch.randn(units, device=G.DEV, generator=g) if act else None
    pooled, y = (torch.full((n, k), -7.0, dtype=torch.float16, device=G.DEV) for k in (c, units))
    B.relay_fused_avgpool_dense(B.RELAY_F16, n, c, hw, units, x, w, b, act, pooled, y)
    torch.cuda.synchronize()
    mean = x.double().mean(1)
    # half a unit of the fp16 result and the fp32 sums (at most hw + 2 roundings of partial sums below hw * max)
    tol = 2.0 ** -11 * mean.abs() + 2.0 ** -24 + (hw + 2) * 2.0 ** -24 * x.double().abs().mean(1)
    assert bool(((pooled.double() - mean).abs() <= tol).all())
    xs, ws = pooled.double().cpu(), w.double().cpu()
    ref, mag = xs @ ws.T, xs.abs() @ ws.abs().T
    if act:
        ref, mag = (ref + b.double().cpu()).clamp(min=0), mag + b.double().cpu().abs()
    tol = 2.0 ** -11 * ref.abs() + 2.0 ** -24 + (c // 64 + 16) * 2.0 ** -24 * mag     # (a lane adds c / 64 products, six sums over lanes)
    assert bool(((y.double().cpu() - ref).abs() <= tol).all())


def test_what_is_refused(G):
    from paper_1904_08368_amd import binding as B
    t = torch.zeros(1 << 16, dtype=torch.float16, device=G.DEV)
    for dt, n, c, hw, units, act in ((B.RELAY_F32, 1, 64, 4, 8, 0), (B.RELAY_F16, 1, 60, 4, 8, 0), (B.RELAY_F16, 1, 2056, 1, 1, 0),
                                     (B.RELAY_F16, 0, 64, 4, 8, 0), (B.RELAY_F16, 1, 64, 4, 8, 2)):
        assert act or not B.relay_avgpool_dense_pays(dt, n, c, hw, units)
        with pytest.raises(B.RelayError):
            B.relay_fused_avgpool_dense(dt, n, c, hw, units, t, t[8192:], None, act, t[16384:], t[32768:])
    for pooled, y in ((t[16384:], t[16384:]), (t[4:], t[32768:]), (t, t[32768:])):
        with pytest.raises(B.RelayError):
            B.relay_fused_avgpool_dense(B.RELAY_F16, 1, 64, 4, 8, t, t[8192:], None, 0, pooled, y)
