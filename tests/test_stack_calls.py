"""FusedNet.run over its list of calls: neighbouring convs in one launch, and a list that its owner has edited."""
import numpy as np
import pytest
import torch

from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet
from workloads import nets


@pytest.fixture
def net(monkeypatch):
    """A network of four calls, of which the second and third share a launch, and what its runs called."""
    done = []
    net = FusedNet.__new__(FusedNet)
    net.side_calls = set()
    net.calls = [(lambda *a, i=i: done.append(i), ("args", i)) for i in range(4)]
    net.pairs = {1: (net.calls[1], net.calls[2])}
    monkeypatch.setattr(B, "relay_conv2d_pair", lambda a, b: done.append((a[1], b[1])))
    return net, done


def test_a_pair_is_one_call(net):
    net, done = net
    net.run()
    assert done == [0, (1, 2), 3]


def test_without_pairs_every_entry_is_called(net):
    net, done = net
    net.pairs = {}
    net.run()
    assert done == [0, 1, 2, 3]


def test_a_wrapped_entry_is_called(net):
    net, done = net
    net.calls[2] = (lambda *a: done.append("wrapped"), net.calls[2][1])
    net.run()
    assert done == [0, 1, "wrapped", 3]


def test_a_shortened_list_and_one_with_an_entry_more(net):
    net, done = net
    net.calls = net.calls[:2]
    net.run()
    assert done == [0, 1]
    done.clear()
    net.calls.insert(0, (lambda *a: done.append("new"), ()))
    net.run()
    assert done == ["new", 0, 1]


def test_the_first_calls_as_one_launch_unless_edited(net):
    net, done = net
    net.stem = (net.calls[:1], lambda *a: done.append(("stem",) + a), ("x",))
    net.run()
    assert done == [("stem", "x"), (1, 2), 3]
    done.clear()
    net.calls[0] = (lambda *a: done.append("edited"), ())
    net.run()
    assert done == ["edited", (1, 2), 3]


def test_calls_with_a_launch_of_their_own_unless_edited(net):
    net, done = net
    net.pairs, net.merged = {}, {2: (net.calls[2:4], lambda *a: done.append(a), ("both",))}
    net.run()
    assert done == [0, 1, ("both",)]
    done.clear()
    net.calls[3] = (lambda *a: done.append("edited"), ())
    net.run()
    assert done == [0, 1, 2, "edited"]


def test_a_forced_tile_or_split_reaches_the_first_conv(net):
    net, done = net
    net.stem = (net.calls[:1], lambda *a: done.append("stem"), ())
    for set_, off, on in ((B.relay_set_conv_tile, -1, -2), (B.relay_set_conv_tile, -1, 5), (B.relay_set_conv_split, 0, 1)):
        set_(on)
        try:
            net.run()
        finally:
            set_(off)
        assert done == [0, (1, 2), 3]
        done.clear()
    net.run()
    assert done == ["stem", (1, 2), 3]


def test_launches_are_what_a_run_makes(net):
    net, done = net
    net.call_names = list("abcd")
    net.stem, net.merged = (net.calls[:1], lambda *a: done.append("stem"), ()), {}
    assert [n for n, _, _ in net.launches()] == ["a", "b+c", "d"]
    for _, fn, args in net.launches():
        fn(*args)
    assert done == ["stem", (1, 2), 3]
    net.side_calls, net.join_before, net.pairs = {2}, {3}, {}
    net.merged = {1: (net.calls[1:3], None, ()), 2: (net.calls[2:4], None, ())}     # across a fork, across a join
    assert [n for n, _, _ in net.launches()] == ["a", "b", "c", "d"]


@pytest.fixture
def built(monkeypatch):
    """FusedNet's constructor without a GPU: what it would launch is left out, what it asks the library is answered."""
    monkeypatch.setattr(B, "relay_prepack_conv2d_weights", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "Stream", lambda **k: object())

    def make(ops, batch, h, w, channels, **kw):
        params = []
        for o in ops:
            p = {"w": np.zeros((o.cout, o.cin, o.r, o.r), np.float16)} if o.kind == "conv" else {}
            if o.bias:
                p["bias"] = np.zeros(o.cout, np.float32)
            if o.bn:
                p["scale"], p["shift"] = np.ones(o.cout, np.float32), np.zeros(o.cout, np.float32)
            params.append(p)
        return FusedNet(ops, params, batch, h, w, "f16", in_channels=channels, device="cpu", **kw)
    return make


def _pool(name, src, c, r, stride, pad):
    return nets.Op("maxpool", name, src, name, cin=c, cout=c, r=r, stride=stride, pad=pad)


def _beside_pool(case):
    """Operators on a tensor that a max pool reads too, listed ahead of that pool, and the names of the launches they share."""
    first = nets.conv("t", "x", "t", 64, 64, 1, 1, 0)
    if case == "pair":
        return [first, nets.conv("a", "t", "a", 64, 128, 3, 2, 1), nets.conv("d", "t", "d", 64, 128, 1, 2, 0, relu=False)], "a+d"
    if case == "conv_and_its_pool":
        return [first, nets.conv("a", "t", "a", 64, 64, 3, 1, 1, bn=False, bias=True), _pool("q", "a", 64, 2, 2, 0)], "a+q"
    return [first, nets.conv("a", "t", "a", 64, 64, 3, 1, 1), nets.conv("b", "a", "b", 64, 64, 3, 1, 1, res="t")], "a+b"


@pytest.mark.parametrize("case,batch,side", [("pair", 1, 28), ("conv_and_its_pool", 8, 112), ("block", 1, 56)])
def test_a_pool_does_not_part_calls_that_share_a_launch(built, case, batch, side):
    """The pool reads what the first of them reads: with and without combine= the launches are the same."""
    ops, shared = _beside_pool(case)
    ops = ops + [_pool("p", "t", 64, 3, 2, 1)]
    names = [[n for n, _, _ in built(ops, batch, side, side, 64, **kw).launches()] for kw in ({}, {"combine": True})]
    assert shared in names[0] and names[1] == names[0]


def test_a_pool_does_not_take_a_fork_away(built):
    ops = _beside_pool("pair")[0] + [_pool("p", "t", 64, 3, 2, 1), nets.conv("c", "a", "c", 128, 128, 3, 1, 1, res="d")]
    two = [built(ops, 1, 28, 28, 64, overlap_shortcuts=True, **kw) for kw in ({}, {"combine": True})]
    assert two[0].side_calls and two[1].call_names == two[0].call_names
    assert (two[1].side_calls, two[1].join_before) == (two[0].side_calls, two[0].join_before)


def test_a_pool_moves_where_that_saves_a_launch(built):
    """An Inception block: the pool beside the convs on its input, and its projection beside the two longer convs; on a few images, where
    nothing shares a launch, the order is the list's."""
    moved, listed = (built(nets.inception_block(), n, 28, 28, 256, combine=True) for n in (32, 2))
    conv, pool, behind = "b1+b3r+b5r", "pool", ["b3", "b5", "bp"]
    assert [n for n, _, _ in moved.launches()] == ["nchw_to_nhwc", conv + "+" + pool, "+".join(behind)]
    assert moved.call_names == ["nchw_to_nhwc", conv, pool] + behind
    assert listed.call_names == ["nchw_to_nhwc", conv] + behind[:2] + [pool] + behind[2:] == [n for n, _, _ in listed.launches()]
