"""The streams that a Rasterizer's workspaces are handed out to."""
import copy
import pickle

import pytest
import torch

from paper_2410_00486_amd import raster


class Workspace:
    device = torch.device("cpu")

    def numel(self):
        return 64


class Plan:
    ws_bytes = 64

    def new_workspace(self, device):
        return Workspace()


@pytest.fixture
def now(monkeypatch):
    """The current stream and whether it is being recorded."""
    state = {"stream": "a", "recording": False}
    monkeypatch.setattr(raster, "_stream_key", lambda: (0, state["stream"]), raising=False)
    monkeypatch.setattr(raster, "_recording", lambda: state["recording"], raising=False)
    return state


def _rasterizer():
    rz = raster.Rasterizer([(8, 8)], 0)
    rz.plan = Plan()
    return rz


def test_a_workspace_stays_with_its_stream(now):
    """A workspace that one stream's kernels may still read goes to no call on
    another stream, and comes back to the next one on its own."""
    rz = _rasterizer()
    ws = rz.acquire("cpu")
    rz.release(rz.plan, ws)
    now["stream"] = "b"
    other = rz.acquire("cpu")
    assert other is not ws
    rz.release(rz.plan, other)
    assert rz.acquire("cpu") is other
    now["stream"] = "a"
    assert rz.acquire("cpu") is ws


def test_the_pool_is_bounded(now):
    """One call each on many streams leaves a bounded number of workspaces; the
    stream's own and those of recorded graphs are all kept."""
    rz = _rasterizer()
    now.update(stream="g", recording=True)
    graphs = rz.acquire("cpu")
    rz.release(rz.plan, graphs)
    now["recording"] = False
    for k in range(40):
        now["stream"] = k
        rz.release(rz.plan, rz.acquire("cpu"))
    assert len(rz._free) <= 2 + 8 and any(ws is graphs for ws in rz._free)
    mine = [rz.acquire("cpu") for _ in range(20)]
    for ws in mine:
        rz.release(rz.plan, ws)
    assert {id(rz.acquire("cpu")) for _ in range(20)} == {id(ws) for ws in mine}


def test_a_recorded_workspace_serves_recordings_on_its_stream(now):
    """A workspace that a graph was recorded with goes to no eager call and to
    no other stream; a recording takes what an eager call left, whatever its
    stream."""
    rz = _rasterizer()
    ws = rz.acquire("cpu")
    rz.release(rz.plan, ws)
    now.update(stream="b", recording=True)
    assert rz.acquire("cpu") is ws
    rz.release(rz.plan, ws)
    now.update(stream="a")
    assert rz.acquire("cpu") is not ws
    now.update(stream="b", recording=False)
    assert rz.acquire("cpu") is not ws
    now.update(recording=True)
    assert rz.acquire("cpu") is ws


def test_a_copied_rasterizer_has_a_pool_of_its_own(now):
    rz = _rasterizer()
    rz.plan, plan = None, rz.plan
    for other in (copy.deepcopy(rz), pickle.loads(pickle.dumps(rz))):
        other.plan = rz.plan = plan
        ws = rz.acquire("cpu")
        rz.release(plan, ws)
        assert other._free == [] and rz._free == [ws]
        rz.plan = None
