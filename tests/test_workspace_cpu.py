"""Which tensor get_workspace hands out, eagerly and under graph capture (host logic only: the allocations are replaced)."""
import pytest

import paper_2402_13533_amd as fhpc

torch = pytest.importorskip("torch")
HEADER = 16384


@pytest.fixture
def device(monkeypatch):
    """A stream that is captured or not as the test says; device memory is host memory that nobody cleared."""
    state = {"capture": 0, "stream": 7}
    empty, zeros = torch.empty, torch.zeros
    monkeypatch.setattr(torch, "empty", lambda n, dtype, device: empty(n, dtype=dtype).fill_(0xFF))
    # work recorded while capturing has not run when the next graph is replayed: a cleared allocation is not clear
    monkeypatch.setattr(torch, "zeros", lambda n, dtype, device: empty(n, dtype=dtype).fill_(0xFF) if state["capture"] else zeros(n, dtype=dtype))
    monkeypatch.setattr(fhpc, "_capturing", lambda: state["capture"] != 0, raising=False)
    monkeypatch.setattr(fhpc, "_raw_stream", lambda index: state["stream"])
    monkeypatch.setattr(fhpc, "_capture_id", lambda stream: state["capture"], raising=False)
    monkeypatch.setattr(fhpc, "_workspaces", {})
    monkeypatch.setattr(fhpc, "_capture_workspaces", {}, raising=False)
    return state


def _get(n):
    return fhpc.get_workspace(n, torch.device("cuda", 0))


def test_every_captured_graph_has_its_own_workspace_and_clears_it(device):
    device["capture"] = 1
    first = _get(20000)
    assert int(first[:HEADER].sum()) == 0 and not fhpc._workspaces
    assert _get(100) is first                                         # the capture's other calls share it
    larger = _get(40000)
    assert larger.numel() >= 40000 and int(larger[:HEADER].sum()) == 0
    device["capture"] = 2                                             # (the first graph may be replayed after this one, or never)
    second = _get(20000)
    assert second is not first and second is not larger
    assert int(second[:HEADER].sum()) == 0 and not fhpc._workspaces
    device["capture"] = 0
    eager = _get(20000)
    assert eager is not second and int(eager.sum()) == 0 and not fhpc._capture_workspaces
    assert _get(300) is eager


def test_a_capture_does_not_take_the_eager_workspace(device):
    """The eager tensor is replaced by a larger one on demand, and the graph would keep its address."""
    eager = _get(20000)
    device["capture"] = 1
    captured = _get(300)
    assert captured is not eager and captured.numel() >= HEADER
    device["stream"] = 8                                              # a forked stream of the same capture
    assert _get(300) is not captured
    device["capture"] = 0
    device["stream"] = 7
    assert _get(300) is eager
