"""Kept workspaces are shared only by calls that run one after the other: those of
one thread on one stream (CPU: the stream query is replaced)."""
import threading

import pytest

torch = pytest.importorskip("torch")

import paper_1801_01473_amd as lq  # noqa: E402

CPU = torch.device("cpu")


@pytest.fixture
def stream(monkeypatch):
    now = [0]
    monkeypatch.setattr(lq, "_stream", lambda: now[0])
    lq.release_workspace()
    yield now
    lq.release_workspace()


def test_one_workspace_per_stream(stream):
    a = lq._workspace(1000, CPU)
    assert lq._workspace(500, CPU).data_ptr() == a.data_ptr()
    stream[0] = 7
    b = lq._workspace(1000, CPU)
    assert b.data_ptr() != a.data_ptr()
    stream[0] = 0
    assert lq._workspace(1000, CPU).data_ptr() == a.data_ptr()
    assert lq._workspace(4000, CPU).numel() >= 4000


def test_one_workspace_per_thread(stream):
    a = lq._workspace(1000, CPU)
    got = []
    t = threading.Thread(target=lambda: got.append(lq._workspace(1000, CPU)))
    t.start()
    t.join()
    assert got[0].data_ptr() != a.data_ptr()


def test_release_and_out_of_memory(stream, monkeypatch):
    """Released for every stream; an allocation that fails is tried again without
    what the other streams keep."""
    lq._workspace(1000, CPU)
    stream[0] = 7
    lq._workspace(1000, CPU)
    lq.release_workspace()
    assert not lq._workspaces()
    lq._workspace(1000, CPU)
    stream[0] = 8
    empty, failed = torch.empty, []

    def limited(n, **k):
        if lq._workspaces():
            failed.append(n)
            raise torch.OutOfMemoryError("limit")
        return empty(n, **k)

    monkeypatch.setattr(torch, "empty", limited)
    ws = lq._workspace(2000, CPU)
    assert failed == [2000] and ws.numel() >= 2000


def test_twice_the_size_is_not_kept(stream, monkeypatch):
    """Twice a size comes from the kept workspace or is given back; without the
    memory for it, the size itself."""
    small = lq._workspace_twice(1000, CPU)
    assert lq._workspace(2000, CPU).data_ptr() == small.data_ptr()
    monkeypatch.setattr(lq, "_KEEP_TWICE", 0)
    lq.release_workspace()
    ws = lq._workspace_twice(1000, CPU)
    assert ws.numel() == 2000 and not lq._workspaces()
    kept = lq._workspace(3000, CPU)
    assert lq._workspace_twice(1000, CPU).data_ptr() == kept.data_ptr()
    lq.release_workspace()
    empty = torch.empty

    def limited(n, **k):
        if n > 1500:
            raise torch.OutOfMemoryError("limit")
        return empty(n, **k)

    monkeypatch.setattr(torch, "empty", limited)
    assert 1000 <= lq._workspace_twice(1000, CPU).numel() < 2000
