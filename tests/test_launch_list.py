"""A captured network's launches enqueued one by one (relay_launch_list_*) against the same network called eagerly: the same bits
on every replay, with new inputs and eager work in between, on other streams and from several threads.  (Every kernel is
deterministic and the launches and their arguments are the same, so the bound is equality.)"""
import ctypes as C
import threading
import time

import numpy as np
import pytest
import torch

from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet
from workloads import inputs, nets


def test_arguments_are_checked_on_the_host():
    out = C.c_void_p(7)
    lib = B.lib()
    assert lib.relay_launch_list_create(None, C.byref(out)) == 1
    assert lib.relay_launch_list_create(0x1000, None) == 1
    assert lib.relay_launch_list_run(None, None) == 1
    assert lib.relay_launch_list_destroy(None) == 1


def _net(name, batch, hw, **kw):
    ops = {"dqn": nets.dqn, "resnet18": nets.resnet18}[name]()
    return FusedNet(ops, inputs.net_params(ops, 5, "f16"), batch, hw, hw, "f16", in_channels=4 if name == "dqn" else 3, **kw), ops[-1].dst


def _inputs(name, batch, hw):
    return [inputs.image(s, batch, 4 if name == "dqn" else 3, hw, hw, "f16") for s in (11, 12, 13)]


@pytest.mark.gpu
@pytest.mark.parametrize("name,batch,hw", [("dqn", 1, 84), ("dqn", 5, 84), ("resnet18", 1, 96), ("resnet18", 3, 61)])
def test_replays_equal_eager_passes(name, batch, hw):
    net, out = _net(name, batch, hw)
    xs = _inputs(name, batch, hw)
    want = []
    for x in xs:
        net.load_input(x)
        net.run()
        want.append(net.tensor(out).copy())
    assert not np.array_equal(want[0], want[1])
    net.capture()
    assert net.launch_list is not None
    side = torch.cuda.Stream()
    for rep in range(2):
        for x, w in zip(xs, want):
            net.load_input(x)
            net.bufs[out].zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(side if rep else torch.cuda.current_stream()):
                for _ in range(3):
                    net.replay()
            torch.cuda.synchronize()
            assert np.array_equal(net.tensor(out), w)
    raised = []

    def passes():
        try:
            for _ in range(20):
                net.replay()
        except Exception as e:      # (a thread's own exception would end the thread and be lost)
            raised.append(e)
    # (that passes do not mix shows in tests/test_launch_list_cpu.py: here they would give the same bits)
    threads = [threading.Thread(target=passes) for _ in range(4)]
    net.bufs[out].zero_()
    torch.cuda.synchronize()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not raised
    assert np.array_equal(net.tensor(out), want[-1])
    net.graph.replay()      # the graph itself stays usable
    torch.cuda.synchronize()
    assert np.array_equal(net.tensor(out), want[-1])


@pytest.mark.gpu
def test_other_graphs_are_replayed_as_graphs():
    side, out = _net("resnet18", 2, 64, overlap_shortcuts=True)      # forks: no chain
    side.load_input(_inputs("resnet18", 2, 64)[0])
    side.run()
    want = side.tensor(out).copy()
    side.capture()
    assert side.launch_list is None
    side.bufs[out].zero_()
    side.replay()
    torch.cuda.synchronize()
    assert np.array_equal(side.tensor(out), want)
    net, out = _net("dqn", 1, 84)
    extra = torch.zeros(8, device=net.dev)
    net.calls.append((lambda: extra.add_(1), ()))                    # a kernel that is not the library's
    net.capture()
    assert net.launch_list is None
    before = extra[0].item()
    net.replay()
    torch.cuda.synchronize()
    assert extra[0].item() == before + 1


@pytest.mark.gpu
def test_a_graph_that_was_reset_is_refused_and_its_list_keeps_its_arguments():
    net, out = _net("dqn", 3, 84)
    net.load_input(_inputs("dqn", 3, 84)[0])
    net.run()
    want = net.tensor(out).copy()
    net.capture()
    recorded = net.launch_list
    net.graph.reset()
    net.bufs[out].zero_()
    with pytest.raises(RuntimeError):
        net.replay()
    torch.cuda.synchronize()
    assert not net.tensor(out).any()
    assert recorded.run()                # (the network's buffers are there; the graph's nodes are not)
    torch.cuda.synchronize()
    assert np.array_equal(net.tensor(out), want)
    with torch.cuda.graph(net.graph):    # another capture into the same object
        net.bufs[out].fill_(3)
    net.replay()
    torch.cuda.synchronize()
    assert (net.tensor(out) == 3).all()
    net.capture()
    net.replay()
    torch.cuda.synchronize()
    assert np.array_equal(net.tensor(out), want)


@pytest.mark.gpu
@pytest.mark.parametrize("name,batch,hw,always", [("dqn", 1, 84, True), ("resnet18", 1, 96, False)])
def test_a_replay_into_a_capture_is_refused_and_the_capture_stays_usable(name, batch, hw, always):
    net, out = _net(name, batch, hw)
    net.load_input(_inputs(name, batch, hw)[0])
    net.capture()
    assert net.list_always == always
    net.replay()
    torch.cuda.synchronize()
    want, mark = net.tensor(out).copy(), torch.zeros(8, device=net.dev)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mark.add_(1)
        for wait in (0.0, 0.001):       # (right behind another pass and later: list and graph)
            time.sleep(wait)
            with pytest.raises(RuntimeError):
                net.replay()
        net.run()
        mark.add_(1)
    for rep in (1, 2):
        net.bufs[out].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert mark[0].item() == 2 * rep and np.array_equal(net.tensor(out), want)
    net.bufs[out].zero_()
    net.replay()
    torch.cuda.synchronize()
    assert np.array_equal(net.tensor(out), want)
