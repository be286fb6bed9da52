"""FusedNet.run over its list of calls: neighbouring convs in one launch, and a list that its owner has edited."""
import pytest

from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet


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
