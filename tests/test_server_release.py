"""Host logic of CCLServer.release (no device): the order of waits, submissions
and the server's end, against stubs that record them.

A released block may be written again, or its memory freed, only after the work
that its caller had enqueued on its stream by then: every server stream waits
for the released blocks' events before the next submission, and before the
server is destroyed (which waits for the server's streams)."""
import collections
import ctypes
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1105_5804_amd import _lib  # noqa: E402
from paper_1105_5804_amd import server as server_module  # noqa: E402
from paper_1105_5804_amd.server import CCLServer  # noqa: E402


class _Stream:
    """handle as a HIP stream, id as torch numbers it (an external stream's is
    its handle)."""

    def __init__(self, handle, stream_id, log):
        self.cuda_stream, self.stream_id, self.log = handle, stream_id, log

    def wait_event(self, ev):
        self.log.append(("wait", self.cuda_stream, ev.recorded))


def _server(monkeypatch, n_streams=2):
    log = []
    current = {}
    serial = iter(range(1000))

    class Event:
        def record(self, stream):
            self.recorded = next(serial)
            log.append(("record", stream.cuda_stream, self.recorded))

    cuda = types.SimpleNamespace(Event=Event, current_stream=lambda device=None: current["stream"])
    monkeypatch.setattr(server_module, "_torch", lambda: types.SimpleNamespace(cuda=cuda))

    def call(name):
        def f(*args):
            log.append((name,))
            return _lib.SW_OK
        return f

    lib = types.SimpleNamespace(**{n: call(n) for n in ("ccl_server_submit", "ccl_server_release",
                                                        "ccl_server_destroy")})
    monkeypatch.setattr(_lib, "lib", lambda: lib)
    srv = object.__new__(CCLServer)
    srv._h = ctypes.c_void_p(1)
    srv.device = None
    srv.streams = [_Stream(1000 + k, 8 * k + 3, log) for k in range(n_streams)]
    srv._fences = {}
    srv._queue = collections.deque()
    srv._inflight = {k: (k, None, 1, 1) for k in range(8)}
    return srv, log, current


def _waited_before(log, name):
    """{server stream: events it waited for} ahead of the last call of `name`."""
    end = max(i for i, e in enumerate(log) if e[0] == name)
    waits = collections.defaultdict(set)
    for e in log[:end]:
        if e[0] == "wait":
            waits[e[1]].add(e[2])
    return waits


def test_close_waits_for_released_blocks(monkeypatch):
    srv, log, current = _server(monkeypatch)
    current["stream"] = _Stream(7, 11, log)
    srv.release(0)
    current["stream"] = _Stream(0, 0, log)
    srv.release(1)
    srv.close()
    waits = _waited_before(log, "ccl_server_destroy")
    assert set(waits) == {1000, 1001} and all(w == {0, 1} for w in waits.values())
    n = len(log)
    srv.close()  # a second close does nothing
    assert len(log) == n


def test_a_run_of_releases_waits_once(monkeypatch):
    srv, log, current = _server(monkeypatch)
    current["stream"] = _Stream(7, 11, log)
    for k in range(4):
        srv.release(k)
    img = torch.zeros((2, 2), dtype=torch.uint8)
    assert srv._try_submit(9, img)
    waits = _waited_before(log, "ccl_server_submit")
    assert all(waits[s] == {3} for s in (1000, 1001))  # the stream's last event covers the ones before it
    n = sum(e[0] == "wait" for e in log)
    assert srv._try_submit(10, img)
    assert sum(e[0] == "wait" for e in log) == n


def test_streams_of_the_caller_keep_every_event(monkeypatch):
    """A caller's own stream may be destroyed and its handle come again: the
    event of a later release there says nothing about the earlier one's work."""
    srv, log, current = _server(monkeypatch)
    for k in range(3):
        current["stream"] = _Stream(4096, 4096, log)
        srv.release(k)
    assert srv._try_submit(9, torch.zeros((2, 2), dtype=torch.uint8))
    waits = _waited_before(log, "ccl_server_submit")
    assert all(waits[s] == {0, 1, 2} for s in (1000, 1001))
