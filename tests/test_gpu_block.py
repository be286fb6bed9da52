"""The two 3x3 convs of a residual block as one launch (relay_fused_conv2d_block, relay_qconv2d_block) against the two separate calls,
bit for bit, and against the oracle; which blocks take it; what the calls refuse."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from oracle.stack import run_float, run_quantized
from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet
from workloads import inputs, nets


def _desc(mode, n, h, w, flags, c=64, k=64):
    return B.conv_desc(n, c, h, w, k, 3, 3, 1, 1, B.RELAY_F16 if mode == "f16" else B.RELAY_I8, B.RELAY_NHWC, flags)


BN, RES, RELU = (B.flags_of(None, *a) for a in ((True, None, False), (None, True, False), (None, None, True)))
BIAS = B.flags_of(True, None, None, False)


def test_which_blocks_take_one_launch():
    """(host only) Up to 256 (int8: 512, and 700 where the convs are past the small-tile kernel) workgroups of 4 x 8 outputs, 64 channels, the first conv
    without a residual."""
    pays = lambda m, n, h, w, f0=BN | RELU, f1=BN | RES | RELU, **k: B.relay_conv2d_block_pays(_desc(m, n, h, w, f0, **k), _desc(m, n, h, w, f1, **k))
    assert pays("f16", 1, 56, 56) and pays("f16", 2, 56, 56) and not pays("f16", 3, 56, 56)
    assert pays("i8", 1, 56, 56, RELU, RES | RELU) and pays("i8", 7, 56, 56, RELU, RES | RELU) and not pays("i8", 8, 56, 56, RELU, RES | RELU)
    i8 = lambda n, h, w: pays("i8", n, h, w, RELU, RES | RELU)
    assert i8(64, 14, 14) and i8(116, 5, 9) and i8(512, 1, 1) and i8(87, 14, 14)
    assert not i8(80, 14, 14) and not i8(32, 13, 33) and not i8(100, 9, 9) and not i8(513, 1, 1)
    assert pays("f16", 1, 7, 64) and pays("f16", 1, 1, 1, BIAS, BIAS)
    assert not pays("f16", 1, 56, 56, RES | RELU) and not pays("f16", 1, 28, 28, c=128, k=128)
    assert not B.relay_conv2d_block_pays(_desc("f16", 1, 56, 56, 0), _desc("f16", 1, 56, 55, 0))
    B.relay_set_conv_tile(10)
    try:
        assert not pays("f16", 1, 56, 56)
    finally:
        B.relay_set_conv_tile(-1)
    with pytest.raises(B.RelayError):
        B.relay_conv2d_block_pays(_desc("f16", 1, 8, 8, 0), _desc("i8", 1, 8, 8, 0))


def test_refused_calls():
    """(host only: every check runs before the first launch)"""
    a = [(1 << 30) + i * (1 << 20) for i in range(12)]
    d0, d1 = _desc("f16", 1, 8, 8, BN), _desc("f16", 1, 8, 8, BN | RES)
    def call(x=a[0], w1=a[1], t=a[2], w2=a[3], y=a[4], sc2=a[7], first=d0, second=d1):
        return B.lib().relay_fused_conv2d_block(C.byref(first) if first else None, x, w1, None, a[5], a[6], t, C.byref(second) if second else None, w2, None,
                                                sc2, a[8], y, None)
    assert call(first=None) == 1 and call(x=None) == 1 and call(t=None) == 1 and call(sc2=None) == 1
    assert call(t=a[0]) == 4 and call(y=a[0]) == 4 and call(y=a[2]) == 4 and call(y=a[1]) == 4 and call(t=a[3]) == 4
    assert call(x=a[0] + 2) == 5 and call(first=_desc("i8", 1, 8, 8, 0)) == 3
    q = lambda s: B.lib().relay_qconv2d_block(C.byref(_desc("i8", 1, 8, 8, 0)), a[0], a[1], None, s, a[2], C.byref(_desc("i8", 1, 8, 8, 0)), a[3], None, 0, 7, a[4], None)
    assert q(32) == 4


def _calls(mode, n, h, w, f0, f1, seed):
    """Arguments of the two separate calls."""
    g = torch.Generator().manual_seed(seed)
    dt = torch.float16 if mode == "f16" else torch.int8
    rnd = (lambda *s: torch.randn(*s, generator=g)) if mode == "f16" else (lambda *s: torch.randint(-127, 128, s, generator=g))
    cuda = lambda t: t.to("cuda")
    x = cuda(rnd(n, h, w, 64).to(dt))
    calls, src = [], x
    for f in (f0, f1):
        d = _desc(mode, n, h, w, f)
        wt = cuda((rnd(64, 64, 3, 3) * (0.06 if mode == "f16" else 1)).to(dt))
        wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
        B.relay_prepack_conv2d_weights(d, wt, 64, wp)
        # (channel ranges that are not 16-byte aligned, and values behind them that must not be read)
        vec = lambda scale, shift: cuda(torch.cat([torch.full((1,), float("nan")), torch.randn(64, generator=g) * scale + shift, torch.full((7,), float("nan"))]))[1:65]
        y = torch.full((n, h, w, 64), 3, dtype=dt, device="cuda")
        res = x if f & RES else None
        if mode == "f16":
            bias, sc, sf = vec(0.1, 0) if f & BIAS else None, vec(0.1, 1) if f & BN else None, vec(0.1, 0) if f & BN else None
            calls.append((d, src, wp, bias, sc, sf, res, y))
        else:
            qb = cuda(torch.randint(-5000, 5000, (64,), generator=g, dtype=torch.int32)) if f & BIAS else None
            calls.append((d, src, wp, qb, res, 9 if f & RES else 0, 11, y))
        src = y
    return calls


def _both(mode, a0, a1):
    t, y = torch.full_like(a0[-1], 5), torch.full_like(a1[-1], 5)
    if mode == "f16":
        B.relay_fused_conv2d_bias_bn_relu(*a0, None)
        B.relay_fused_conv2d_bias_bn_relu(*a1, None)
        B.relay_fused_conv2d_block(*a0[:6], t, a1[0], *a1[2:6], y)
    else:
        B.relay_qconv2d_requant(*a0, None)
        B.relay_qconv2d_requant(*a1, None)
        B.relay_qconv2d_block(*a0[:4], a0[6], t, a1[0], a1[2], a1[3], a1[5], a1[6], y)
    torch.cuda.synchronize()
    return t, y


@pytest.mark.gpu
@pytest.mark.parametrize("mode,f0,f1", [("f16", BN | RELU, BN | RES | RELU), ("f16", BIAS, BIAS | BN | RES), ("f16", 0, 0), ("i8", RELU, RES | RELU), ("i8", BIAS, BIAS)])
def test_bits_of_the_two_calls_at_the_edges(mode, f0, f1):
    """Images of less than a rectangle, of whole ones, of remainders in both directions, one pixel, a row and a column; several images;
    the last size that one launch takes and one beyond it (two launches)."""
    for i, (n, h, w) in enumerate([(1, 1, 1), (1, 4, 8), (1, 5, 9), (2, 3, 17), (1, 64, 1), (1, 1, 64), (3, 8, 16), (2, 13, 7), (1, 56, 56), (2, 56, 56), (7, 56, 56), (8, 56, 56)]):
        a0, a1 = _calls(mode, n, h, w, f0, f1, 700 + i)
        t, y = _both(mode, a0, a1)
        assert torch.equal(t.view(torch.uint8), a0[-1].view(torch.uint8)), (mode, n, h, w, "first")
        assert torch.equal(y.view(torch.uint8), a1[-1].view(torch.uint8)), (mode, n, h, w, "second")


@pytest.mark.gpu
def test_infinities_reach_what_they_reach_in_the_two_calls():
    a0, a1 = _calls("f16", 1, 9, 19, BN, BN | RES, 31)
    a0[1][0, 4, 9, 3], a0[1][0, 0, 0, 5], a0[1][0, 8, 18, 0] = float("inf"), float("-inf"), float("nan")
    t, y = _both("f16", a0, a1)
    assert not torch.isfinite(a1[-1]).all() and torch.isfinite(a1[-1]).any()
    for got, want in ((t, a0[-1]), (y, a1[-1])):
        assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.nan_to_num(got), torch.nan_to_num(want))


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["f16", "i8"])
def test_outputs_that_overlap_an_operand_are_those_of_the_calls_in_order(mode):
    """The second conv's output a few rows into the first one's input (which no residual needs again), and a little ahead of it; for the paired
    call the second member's output in the first one's input, whose launch is the earlier one."""
    n, h, w = 1, 24, 24
    f = RELU
    a0, a1 = _calls(mode, n, h, w, f, f, 77)
    a2 = _calls(mode, n, h, w, f, f, 78)[0]
    row, rows = w * 64, n * h * w * 64
    for shift in (3 * row, -2 * row):
        buf = torch.empty(rows + 3 * row, dtype=a0[1].dtype, device="cuda")
        x0, y0 = max(0, -shift), max(0, shift)
        x, y = buf[x0:x0 + rows].view_as(a0[1]), buf[y0:y0 + rows].view_as(a0[1])
        b0, b1, t = (a0[0], x, *a0[2:]), (*a1[:-1], y), torch.empty_like(x)
        conv, tail = (B.relay_fused_conv2d_bias_bn_relu, 6) if mode == "f16" else (B.relay_qconv2d_requant, 4)
        assert b1[tail] is None and B.relay_conv2d_block_pays(b0[0], b1[0])
        pair = (*a2[:-1], y)   # (reads its own tensor)
        block = (*b0[:6], t, b1[0], *b1[2:6], y) if mode == "f16" else (*b0[:4], b0[6], t, b1[0], b1[2], b1[3], b1[5], b1[6], y)
        ways = ((lambda: (conv(*b0[:-1], t, None), conv(b1[0], t, *b1[2:], None)), lambda: (B.relay_fused_conv2d_block if mode == "f16" else B.relay_qconv2d_block)(*block)),
                (lambda: (conv(*b0[:-1], t, None), conv(*pair, None)), lambda: B.relay_conv2d_pair((*b0[:-1], t, None), (*pair, None))))
        for two, one in ways:
            got = []
            for call in (two, one):
                buf.fill_(1), t.fill_(5), x.copy_(a0[1])
                call()
                torch.cuda.synchronize()
                got.append([v.cpu().view(torch.uint8) for v in (buf, t)])
            assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["f16", "i8"])
def test_a_network_of_one_block(mode):
    """FusedNet takes it: against the oracle, and the same bits as its calls one by one; an edited list of calls is followed."""
    ops = nets.basic_block(64)
    x, params = inputs.image(2, 1, 64, 13, 22, mode), inputs.net_params(ops, 2, mode)
    sh = [{"s": inputs.default_out_rshift(576), "l": inputs.default_out_rshift(576)} for _ in ops] if mode == "i8" else None
    net = FusedNet(ops, params, 1, 13, 22, mode, shifts=sh, in_channels=64)
    assert [n for n, _, _ in net.launches()] == [net.call_names[0], "+".join(net.call_names[1:])]
    net.load_input(x)
    net.run()
    got = {o.dst: net.tensor(o.dst) for o in ops}
    if mode == "f16":
        ref = run_float(ops, params, x, "f16")
        assert max(oracle.max_rel_err(got[o.dst], ref[o.dst]) for o in ops) <= 1e-2
    else:
        ref = run_quantized(ops, params, sh, x)
        assert all(np.array_equal(got[o.dst], ref[o.dst]) for o in ops)
    for fn, args in net.calls:
        fn(*args)
    assert all(np.array_equal(got[o.dst], net.tensor(o.dst)) for o in ops)
    net.bufs[ops[-1].dst].fill_(1)
    net.calls = net.calls[:2]
    net.run()
    assert bool((net.bufs[ops[-1].dst] == 1).all()) and np.array_equal(net.tensor(ops[0].dst), got[ops[0].dst])
