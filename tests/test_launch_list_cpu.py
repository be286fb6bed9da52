"""The launch list on the host: its native part against stand-ins for the HIP calls it makes (tests/launch_list_stub.cpp), and
which of list and graph FusedNet.replay() takes."""
import os
import shutil
import subprocess
import threading

import pytest

from paper_1904_08368_amd import binding as B
from paper_1904_08368_amd.stack import FusedNet

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("launch_list") / "harness")
    r = subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-o", exe,
                        os.path.join(ROOT, "tests", "launch_list_stub.cpp"),
                        os.path.join(ROOT, "paper_1904_08368_amd", "csrc", "launch_list.cpp"), "-ldl", "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("scenario", ["lifetime", "threads", "capture", "device", "refused"])
def test_native_part(harness, scenario):
    """A graph destroyed before its list, passes of four threads, a stream that is being captured, another current device, graphs
    that are no chain of the library's kernels."""
    r = subprocess.run([harness, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr


class _Graph:
    """Stands in for a captured graph: replay() is an error while it holds nothing, as torch's is."""

    def __init__(self):
        self.held, self.holds, self.replays = 0, True, 0

    def reset(self):
        self.held, self.holds = self.held + 1, False

    def replay(self):
        if not self.holds:
            raise RuntimeError("replay without a preceding successful capture")
        self.replays += 1


def _net():
    net = FusedNet.__new__(FusedNet)
    net.graph = _Graph()
    recorded = B.LaunchList.__new__(B.LaunchList)
    recorded.graph, recorded.held, recorded.handle, recorded.runs = net.graph, 0, None, 0

    def run():
        recorded.runs += 1
        return True
    recorded.run = run
    net.launch_list = recorded
    return net, recorded


def test_a_graph_that_was_reset_is_not_replayed():
    net, recorded = _net()
    net.replay()
    assert (recorded.runs, net.graph.replays) == (1, 0)
    net.graph.reset()
    with pytest.raises(RuntimeError):
        net.replay()
    net.graph.holds = True          # another capture into the same object
    net.replay()
    assert (recorded.runs, net.graph.replays) == (1, 1)
    net.graph = _Graph()            # another graph in its place
    net.replay()
    assert (recorded.runs, net.graph.replays) == (1, 1)


def test_a_replay_into_a_capture_is_refused_without_touching_the_graph():
    """(the graph is not instantiated while there is a list, and its first replay would do that inside the caller's capture)"""
    net, recorded = _net()
    recorded.run = lambda: False
    with pytest.raises(RuntimeError):
        net.replay()
    assert net.graph.replays == 0


def test_passes_of_many_short_launches_take_the_list_only_behind_another_pass(monkeypatch):
    from paper_1904_08368_amd import stack
    now = [1_000_000]
    monkeypatch.setattr(stack.time, "perf_counter_ns", lambda: now[0])
    net, recorded = _net()
    net._enqueued = threading.local()
    net.list_always = False
    taken = []
    for gap_us in (1000, 2, 9, 11, 9, 300):
        now[0] += gap_us * 1000
        before = recorded.runs
        net.replay()
        taken.append(recorded.runs - before)
    assert taken == [0, 1, 1, 0, 1, 0] and net.graph.replays == 3
    net.list_always = True
    net.replay()
    assert recorded.runs == 4
