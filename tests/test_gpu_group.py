"""Convs of different inputs into channel segments as one launch (relay_fused_conv2d_combined_group), and one beside a max pool
(relay_fused_conv2d_combined_maxpool), against the separate calls, bit for bit; which
convs take it; what the call refuses; the Inception block that uses it."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet
from workloads import nets

MEMBERS = {"3": (128, 192, 3, 128), "5": (32, 96, 5, 320), "1": (256, 64, 1, 416)}   # channels, filters, window, first channel of 480


def _desc(n, h, w, kind, flags):
    c, k, r, _ = MEMBERS[kind]
    return B.conv_desc(n, c, h, w, k, r, r, 1, r // 2, B.RELAY_F16, B.RELAY_NHWC, flags)


class Address:
    """What a host-only call takes for a tensor."""
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


def _host_members(n, h, w, kinds):
    f = B.flags_of(None, True, None, True)
    at = lambda i, j: Address((i + 1 << 36) + (j << 34))
    return [(_desc(n, h, w, kd, f), at(i, 0), MEMBERS[kd][0], at(i, 1), None, at(i, 2), at(i, 2), [MEMBERS[kd][1]],
             [Address((1 << 40) + 2 * MEMBERS[kd][3] + 960 * 64 * i)], [480]) for i, kd in enumerate(kinds)]


def test_which_convs_share_a_launch():
    """(host only) Convs that take tiles of 128 x 64 or less of the two staged kernels by themselves, one of each kind."""
    pays = lambda n, h, w, kinds: B.relay_conv2d_combined_group_pays(*_host_members(n, h, w, kinds))
    assert all(pays(32, 28, 28, k) for k in ("351", "35", "51", "31", "513", "15")) and pays(12, 28, 28, "351")
    assert not pays(10, 28, 28, "351")                                # (the 5x5 conv runs on the small-tile kernel)
    assert not pays(32, 28, 28, "33") and not pays(32, 28, 28, "11")  # (two of a kind)
    assert not pays(32, 40, 40, "31") and pays(32, 40, 40, "51")      # (a halo too wide for two workgroups a CU)
    assert not pays(32, 64, 64, "51") and not pays(32, 64, 64, "31")  # (wider tiles)
    B.relay_set_conv_tile(9)
    try:
        assert not pays(32, 28, 28, "351")
    finally:
        B.relay_set_conv_tile(-1)


def test_which_widths_share_a_launch():
    """(host only) Both sides of the rule's lines: a long reduction on few tiles, such a one behind more tiles than start at once, short reductions over many pixels."""
    def pays(n, h, w, *members):
        f, out = B.flags_of(None, True, None, True), []
        for i, (c, k, r, s) in enumerate(members):
            at = lambda j: Address((i + 1 << 36) + (j << 34))
            out.append((B.conv_desc(n, c, h, w, k, r, r, s, r // 2, B.RELAY_F16, B.RELAY_NHWC, f), at(0), c, at(1), None, at(2), at(2), [k], [at(3)], [k]))
        return B.relay_conv2d_combined_group_pays(*out)
    short = (32, 64, 1, 1)
    assert pays(8, 28, 28, short, (1600, 64, 1, 1)) and not pays(8, 28, 28, short, (2048, 64, 1, 1)) and not pays(8, 28, 28, short, (512, 64, 3, 2))
    assert pays(16, 28, 28, short, (64, 96, 5, 1)) and not pays(8, 28, 28, short, (256, 96, 5, 1)) and pays(16, 28, 28, short, (256, 96, 5, 1))
    assert pays(32, 17, 17, (96, 96, 5, 1), (256, 64, 1, 1))                    # (long, but not the member whose tiles start last)
    assert pays(13, 27, 31, (128, 192, 3, 1), (256, 96, 5, 1)) and not pays(16, 28, 28, (128, 192, 3, 1), (256, 96, 5, 1))
    assert pays(40, 32, 32, (96, 64, 1, 1), (128, 64, 3, 2)) and not pays(58, 32, 32, (96, 64, 1, 1), (128, 64, 3, 2)) and pays(58, 32, 32, (96, 64, 1, 1), (832, 64, 1, 2))
    assert pays(16, 28, 28, (128, 192, 3, 1), (160, 64, 1, 1), (64, 96, 5, 1)) and not pays(16, 28, 28, (128, 192, 3, 1), (160, 64, 1, 1), (128, 96, 5, 1))
    assert not pays(36, 52, 72, (32, 8, 1, 1), (64, 24, 1, 1)) and not pays(40, 56, 56, short, (64, 64, 1, 1)) and pays(20, 56, 56, short, (64, 64, 1, 1))


def test_refused_calls():
    """(host only: every check runs before the first launch)"""
    def status(members, n=None):
        calls, keep = B._views_calls(members)
        return B.lib().relay_fused_conv2d_combined_group(C.addressof(calls) if members else None, len(members) if n is None else n, None)
    good = _host_members(32, 28, 28, "351")
    swap = lambda i, j, v: [tuple(v if (a, b) == (i, j) else x for b, x in enumerate(m)) for a, m in enumerate(good)]
    assert status([], 2) == 1 and status(good[:1]) == 2 and status(good, 4) == 2
    assert status(swap(1, 1, None)) == 1 and status(swap(2, 5, None)) == 1
    assert status(swap(0, 8, good[1][8])) == 4                        # (one address)
    assert status(swap(1, 1, good[0][8][0])) == 4 and status(swap(2, 3, good[1][8][0])) == 4
    assert status(swap(1, 1, Address(good[1][1].at + 2))) == 5
    assert status(swap(1, 9, [90])) == 2


def _views(n, h, w, cat, spans):
    """Members 5x5 and 1x1 on channel ranges of one tensor of 1024 channels: (first input channel, first output channel) of each; None: a tensor of its own."""
    f, out = B.flags_of(None, True, None, True), []
    for i, (kd, (x0, y0)) in enumerate(zip("51", spans)):
        (c, k, _, _), own = MEMBERS[kd], lambda j: Address((i + 1 << 36) + (j << 34))
        x, x_ld = (own(0), c) if x0 is None else (Address(cat + 2 * x0), 1024)
        y, y_ld = (own(3), k) if y0 is None else (Address(cat + 2 * y0), 1024)
        out.append((_desc(n, h, w, kd, f), x, x_ld, own(1), None, own(2), own(2), [k], [y], [y_ld]))
    return out


def test_members_that_meet_in_memory_keep_their_order():
    """(host only) An output that begins inside another member's input or output view is a dependence though no two addresses are equal; ranges of
    one tensor without a common channel are none, nor are neighbours in one allocation."""
    cat, n, h, w = 1 << 40, 32, 28, 28
    pays = lambda *spans: B.relay_conv2d_combined_group_pays(*_views(n, h, w, cat, spans))
    assert pays((None, None), (None, None)) and pays((None, 0), (None, 96)) and pays((0, 32), (128, 384)) and pays((992, 0), (96, 352))
    assert not pays((None, 64), (0, None))            # 5x5 -> channels 64 .. 159, the 1x1 conv reads 0 .. 255
    assert not pays((80, None), (None, 64))           # 1x1 -> channels 64 .. 127, the 5x5 conv reads 80 .. 111
    assert not pays((None, 0), (None, 88)) and not pays((None, 88), (None, 32))
    members = _views(n, h, w, cat, ((None, None), (None, None)))
    spot = lambda i, at: [tuple([Address(at)] if (a, b) == (i, 8) else x for b, x in enumerate(m)) for a, m in enumerate(members)]
    w1 = members[1][3].at
    assert not B.relay_conv2d_combined_group_pays(*spot(0, w1 + 32)) and not B.relay_conv2d_combined_group_pays(*spot(0, members[1][5].at - 64))
    ends = w1 + B.relay_packed_weight_bytes(members[1][0])
    assert B.relay_conv2d_combined_group_pays(*spot(0, ends)) and not B.relay_conv2d_combined_group_pays(*spot(0, ends - 16))
    # beside a pool
    at = lambda i: (i + 1) << 36
    d, size = B.conv_desc(n, 256, h, w, 288, 1, 1, 1, 0, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(True, None, None, True)), n * h * w * 512
    conv = lambda x, y, ld=288: (d, Address(x), 256, Address(at(1)), Address(at(2)), None, None, [288], [Address(y)], [ld])
    pays = lambda c, x, y: B.relay_conv2d_combined_maxpool_pays(c, _pool_call(n, h, w, 1, Address(x), Address(y)))
    assert pays(conv(at(0), at(3)), at(0), at(4)) and pays(conv(at(0), at(3)), at(0), at(0) + size) and pays(conv(at(0), at(3)), at(0), at(0) - size)
    assert not pays(conv(at(0), at(5) + 128, 512), at(5), at(4))      # the conv stores into the pool's input,
    assert not pays(conv(at(0), at(4) + 64, 512), at(0), at(4))       # into its output,
    assert not pays(conv(at(0), at(3)), at(5), at(0) + 16)            # the pool into the conv's input,
    assert not pays(conv(at(0), at(3)), at(0), at(2) + 16 - size)     # into its bias


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,kinds", [(32, 28, 28, "351"), (12, 28, 28, "315"), (13, 27, 31, "35"), (20, 33, 29, "51"), (20, 33, 29, "31"), (4, 64, 64, "35"),
                                         (10, 28, 28, "351"), (2, 9, 11, "513")])
@pytest.mark.parametrize("tail", ["bn_relu", "bias"])
def test_group_is_the_separate_calls(n, h, w, kinds, tail):
    """Tiles with and without a remainder, one kind absent, and shapes that run as separate launches (the last two)."""
    g = torch.Generator().manual_seed(5)
    flags = B.flags_of(None, True, None, True) if tail == "bn_relu" else B.flags_of(True, None, None, False)
    cat = torch.empty((n, h, w, 480), dtype=torch.float16, device="cuda")
    members = []
    for kind in kinds:
        c, k, r, at = MEMBERS[kind]
        d = _desc(n, h, w, kind, flags)
        x = torch.randn((n, h, w, c), generator=g).half().cuda()
        src = (torch.randn((k, c, r, r), generator=g) * (2.0 / (c * r * r)) ** 0.5).half().cuda()
        wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
        B.relay_prepack_conv2d_weights(d, src, c, wp)
        v = [torch.randn(k, generator=g).cuda() for _ in range(3)]
        members.append((d, x, c, wp) + ((None, v[0], v[1]) if tail == "bn_relu" else (v[2], None, None)) + ([k], [cat[..., at:at + k]], [480]))
    assert B.relay_conv2d_combined_group_pays(*members) == (n > 2 and (n, h, w) != (10, 28, 28))
    got = []
    for call in (lambda: [B.relay_fused_conv2d_combined(*m) for m in members], lambda: B.relay_fused_conv2d_combined_group(*members)):
        cat.fill_(7.0)
        call()
        torch.cuda.synchronize()
        got.append(cat.cpu().view(torch.int16))
    assert torch.equal(got[0], got[1])
    assert torch.isfinite(cat).all() and not (got[0][..., MEMBERS[kinds[0]][3]] == got[0].new_full((), 0x4700)).all()


# (channels, those of the tensor they are in, filters, window, output segments) of each member
VIEWS = {"ranges": ((20, 33, 29), [(32, 96, 96, 5, [24, 8, 56, 8]), (256, 480, 64, 1, [8, 56])]),
         "3x3_of_a_range": ((32, 28, 28), [(128, 192, 192, 3, [72, 104, 16]), (32, 32, 96, 5, [96])]),
         "all_three": ((13, 27, 31), [(128, 128, 200, 3, [40, 160]), (32, 64, 96, 5, [88, 8]), (256, 320, 72, 1, [8, 8, 8, 48])]),
         "filters_larger_than_inputs": ((2, 27, 29), [(128, 128, 776, 3, [776]), (32, 32, 1032, 3, [1000, 32]), (128, 136, 2056, 1, [2056])])}


def _view_members(case, tensor):
    """Arguments of the members, the inputs among NaNs, the constants at odd places (not 16-byte aligned) with a NaN on either side.  tensor(shape, scale)."""
    (n, h, w), members, out, keep = *VIEWS[case], [], []
    flags = B.flags_of(True, True, None, True)
    for c, ld, k, r, segments in members:
        d = B.conv_desc(n, c, h, w, k, r, r, 1, r // 2, B.RELAY_F16, B.RELAY_NHWC, flags)
        wide, x0 = torch.full((n, h, w, ld), float("nan"), dtype=torch.float16, device="cuda"), (ld - c) // 16 * 8
        wide[..., x0:x0 + c] = tensor((n, h, w, c), 1).half()
        wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
        B.relay_prepack_conv2d_weights(d, tensor((k, c, r, r), (2.0 / (c * r * r)) ** 0.5).half(), c, wp)
        bias, scale, shift = (torch.nn.functional.pad(tensor((k,), 1), (1, 2), value=float("nan"))[1:k + 1] for _ in range(3))
        ys = [torch.empty((n, h, w, width + 16 * (i % 2)), dtype=torch.float16, device="cuda") for i, width in enumerate(segments)]
        keep += ys
        out.append((d, wide[..., x0:], ld, wp, bias, scale, shift, segments, [y[..., 8 * (i % 2):] for i, y in enumerate(ys)], [y.shape[3] for y in ys]))
    return out, keep


@pytest.mark.gpu
@pytest.mark.parametrize("case", VIEWS)
def test_group_of_views_is_the_separate_calls(case):
    """Members that read a channel range of a wider tensor (a 3x3 one then runs on the implicit GEMM's tiles), that store into two to four segments which
    end inside a tile, with constants that are not 16-byte aligned, and with filters larger than their inputs (the other order of tiles)."""
    g = torch.Generator().manual_seed(17)
    members, ys = _view_members(case, lambda shape, scale: (torch.randn(shape, generator=g) * scale).cuda())
    assert B.relay_conv2d_combined_group_pays(*members)
    got = []
    for call in (lambda: [B.relay_fused_conv2d_combined(*m) for m in members], lambda: B.relay_fused_conv2d_combined_group(*members)):
        for y in ys:
            y.fill_(7.0)
        call()
        torch.cuda.synchronize()
        got.append([y.cpu() for y in ys])
    for alone, together in zip(*got):
        assert torch.isfinite(alone).all() and torch.equal(alone.view(torch.int16), together.view(torch.int16))


def _pool_call(n, h, w, stride, x, y, r=3, c=256):
    return (B.RELAY_F16, n, c, h, w, r, stride, 1, x, y)


def test_which_convs_share_a_launch_with_a_pool():
    """(host only) Convs on small-ring 128 x 64 tiles by themselves, 3 x 3 windows, at most 200 MiB in all; what is refused."""
    def members(n, h, w, k=288, r=3, stride=1):
        at = lambda i: Address((i + 1) << 36)
        d = B.conv_desc(n, 256, h, w, k, 1, 1, 1, 0, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(True, None, None, True))
        return (d, at(0), 256, at(1), at(2), None, None, [k], [at(3)], [k]), _pool_call(n, h, w, stride, at(0), at(4), r)
    pays = lambda *a, **k: B.relay_conv2d_combined_maxpool_pays(*members(*a, **k))
    assert pays(32, 28, 28) and pays(17, 28, 28) and pays(32, 28, 28, stride=2) and pays(32, 64, 64)
    assert not pays(3, 17, 40) and not pays(16, 28, 28) and not pays(32, 28, 28, r=2)
    assert pays(32, 56, 56, k=512) and not pays(32, 56, 56, k=544) and pays(32, 56, 56, k=640, stride=2)   # 196, 202, 184 MiB
    conv, pool = members(32, 56, 56, k=448)
    assert B.relay_conv2d_combined_maxpool_pays(conv, pool) and not B.relay_conv2d_combined_maxpool_pays(conv, (*pool[:8], Address(9 << 36), pool[9]))
    B.relay_set_conv_split(2)
    try:
        assert not pays(32, 28, 28)
    finally:
        B.relay_set_conv_split(0)
    conv, pool = members(32, 28, 28)
    for i, bad in ((9, pool[8]), (8, conv[8][0]), (9, conv[8][0]), (9, conv[3])):
        with pytest.raises(B.RelayError, match="UNSUPPORTED"):
            B.relay_conv2d_combined_maxpool_pays(conv, tuple(bad if j == i else v for j, v in enumerate(pool)))
    with pytest.raises(B.RelayError, match="SHAPE"):
        B.relay_conv2d_combined_maxpool_pays(conv, _pool_call(32, 28, 28, 0, pool[8], pool[9]))
    with pytest.raises(B.RelayError, match="NULL"):
        B.relay_conv2d_combined_maxpool_pays(conv, _pool_call(32, 28, 28, 1, None, pool[9]))


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,k,stride,c", [(32, 28, 28, 288, 1, 256), (20, 33, 29, 288, 1, 256), (32, 28, 28, 192, 2, 256), (13, 31, 37, 288, 2, 64),
                                              (9, 50, 23, 448, 1, 8), (34, 17, 11, 704, 1, 264), (64, 14, 14, 1024, 1, 256), (46, 21, 17, 256, 2, 1016),
                                              (3, 17, 40, 288, 1, 256)])
def test_conv_and_pool_are_the_separate_calls(n, h, w, k, stride, c):
    """One and two outputs a thread, more workgroups of one and of the other, as many of both, remainders, a NaN and infinities in the pool's input, a pool of another
    tensor; the last runs as two launches."""
    g = torch.Generator().manual_seed(n)
    x = torch.randn((n, h, w, 256), generator=g).half().cuda()
    px = x if c == 256 else torch.randn((n, h, w, c), generator=g).half().cuda()
    if c != 256:
        px[0, 1, 1, :3] = torch.tensor([float("nan"), float("inf"), float("-inf")])
    d = B.conv_desc(n, 256, h, w, k, 1, 1, 1, 0, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(True, None, None, True))
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
    B.relay_prepack_conv2d_weights(d, (torch.randn((k, 256, 1, 1), generator=g) / 16).half().cuda(), 256, wp)
    y = torch.empty((n, h, w, k), dtype=torch.float16, device="cuda")
    py = torch.empty((n, (h - 1) // stride + 1, (w - 1) // stride + 1, c), dtype=torch.float16, device="cuda")
    conv, pool = (d, x, 256, wp, torch.randn(k, generator=g).cuda(), None, None, [k], [y], [k]), _pool_call(n, h, w, stride, px, py, c=c)
    assert B.relay_conv2d_combined_maxpool_pays(conv, pool) == (n > 3)
    got = []
    for call in (lambda: (B.relay_fused_conv2d_combined(*conv), B.relay_maxpool2d(*pool)), lambda: B.relay_fused_conv2d_combined_maxpool(conv, pool)):
        y.fill_(7.0), py.fill_(7.0)
        call()
        torch.cuda.synchronize()
        got.append([t.cpu().view(torch.int16) for t in (y, py)])
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.gpu
def test_conv_of_a_range_and_pool_are_the_separate_calls():
    """The conv reads half the channels of the tensor that the pool takes whole, and stores into three segments that end inside a tile; constants not aligned."""
    n, h, w, segments, g = 16, 29, 31, [96, 8, 184], torch.Generator().manual_seed(23)
    wide = torch.randn((n, h, w, 512), generator=g).half().cuda()
    d = B.conv_desc(n, 256, h, w, 288, 1, 1, 1, 0, B.RELAY_F16, B.RELAY_NHWC, B.flags_of(None, True, None, True))
    wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
    B.relay_prepack_conv2d_weights(d, (torch.randn((288, 256, 1, 1), generator=g) / 16).half().cuda(), 256, wp)
    scale, shift = (torch.nn.functional.pad(torch.randn(288, generator=g), (1, 3), value=float("nan")).cuda()[1:289] for _ in range(2))
    ys = [torch.empty((n, h, w, k + 8), dtype=torch.float16, device="cuda") for k in segments]
    py = torch.empty_like(wide)
    conv = (d, wide[..., 128:], 512, wp, None, scale, shift, segments, [y[..., 8:] for y in ys], [y.shape[3] for y in ys])
    pool = _pool_call(n, h, w, 1, wide, py, c=512)
    assert B.relay_conv2d_combined_maxpool_pays(conv, pool)
    got = []
    for call in (lambda: (B.relay_fused_conv2d_combined(*conv), B.relay_maxpool2d(*pool)), lambda: B.relay_fused_conv2d_combined_maxpool(conv, pool)):
        for y in (*ys, py):
            y.fill_(7.0)
        call()
        torch.cuda.synchronize()
        got.append([y.cpu() for y in (*ys, py)])
    for alone, together in zip(*got):
        assert torch.isfinite(alone).all() and torch.equal(alone.view(torch.int16), together.view(torch.int16))


@pytest.mark.gpu
def test_inception_block_runs_them_together():
    """Eager and captured, against the same network with every call by itself, on two inputs."""
    ops, rng = nets.inception_block(), np.random.default_rng(3)
    params = []
    for op in ops:
        p = {}
        if op.kind == "conv":
            p["w"] = (rng.standard_normal((op.cout, op.cin, op.r, op.r)) * np.sqrt(2.0 / (op.cin * op.r * op.r))).astype(np.float16)
            if op.bias:
                p["bias"] = rng.standard_normal(op.cout).astype(np.float32)
            if op.bn:
                p["scale"], p["shift"] = (rng.standard_normal(op.cout).astype(np.float32) for _ in range(2))
        params.append(p)
    net = FusedNet(ops, params, 17, 28, 28, "f16", in_channels=256, combine=True)
    assert {B.relay_fused_conv2d_combined_group, B.relay_fused_conv2d_combined_maxpool} <= {fn for _, fn, _ in net.launches()}
    out = ops[-1].dst
    for seed in range(2):
        net.load_input(np.random.default_rng(seed).standard_normal((17, 256, 28, 28)).astype(np.float16))
        merged, net.merged = net.merged, {}
        net.run()
        alone = net.tensor(out)
        net.merged = merged
        net.bufs[out].fill_(7.0)
        net.run()
        assert np.array_equal(alone.view(np.int16), net.tensor(out).view(np.int16))
        if net.graph is None:
            net.capture()
        for _ in range(3):
            net.bufs[out].fill_(7.0)
            net.replay()
            assert np.array_equal(alone.view(np.int16), net.tensor(out).view(np.int16))


@pytest.mark.gpu
def test_members_that_meet_in_memory_give_what_the_calls_in_order_give():
    """The second conv, or the pool, reads channels that the first conv writes."""
    n, h, w, g = 32, 28, 28, torch.Generator().manual_seed(9)
    wide = torch.randn((n, h, w, 512), generator=g).half().cuda()
    f = B.flags_of(True, None, None, False)

    def member(c, k, r, x, y):
        d = B.conv_desc(n, c, h, w, k, r, r, 1, r // 2, B.RELAY_F16, B.RELAY_NHWC, f)
        wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
        B.relay_prepack_conv2d_weights(d, (torch.randn((k, c, r, r), generator=g) * (2.0 / (c * r * r)) ** 0.5).half().cuda(), c, wp)
        return (d, x, x.stride(2), wp, torch.randn(k, generator=g).cuda(), None, None, [k], [y], [y.stride(2)])
    cat, y1, py = torch.empty_like(wide), torch.empty((n, h, w, 64), dtype=torch.float16, device="cuda"), torch.empty_like(wide)
    first = member(32, 96, 5, torch.randn((n, h, w, 32), generator=g).half().cuda(), cat[..., 64:160])
    second = member(256, 64, 1, cat[..., :256], y1)
    trio = member(256, 288, 1, torch.randn((n, h, w, 256), generator=g).half().cuda(), cat[..., 128:416])
    pool = _pool_call(n, h, w, 1, cat, py, c=512)
    for a, b, one in ((lambda: B.relay_fused_conv2d_combined(*first), lambda: B.relay_fused_conv2d_combined(*second),
                       lambda: B.relay_fused_conv2d_combined_group(first, second)),
                      (lambda: B.relay_fused_conv2d_combined(*trio), lambda: B.relay_maxpool2d(*pool), lambda: B.relay_fused_conv2d_combined_maxpool(trio, pool))):
        got = []
        for call in (lambda: (a(), b()), one):
            cat.copy_(wide), y1.fill_(7.0), py.fill_(7.0)
            call()
            torch.cuda.synchronize()
            got.append([t.cpu().view(torch.int16) for t in (cat, y1, py)])
        assert all(torch.equal(p, q) for p, q in zip(*got))
