"""A backlog (`run(..., realtime=False)`): the drawing of its data is part of
every latency, overlaps over the workers' threads and keeps the order of the
requests."""
import threading
import time

from paper_2002_04894_amd import serve

from test_serve import SYNTH, FakeServer, _fake_torch


def test_backlog_clock_includes_the_drawing(monkeypatch):
    monkeypatch.setattr(serve.fmm, "fmm_bytes_estimate", lambda n, l, th, p: 1)
    seen, lock = [], threading.Lock()

    def draw(r):
        time.sleep(0.05)
        with lock:
            seen.append((r.rid, threading.get_ident()))
        return r.rid

    monkeypatch.setattr(serve, "request_points", draw)
    _fake_torch(monkeypatch)

    class Server(FakeServer):
        def solve(self, req, data, stream, reserve=None):
            assert data == req.rid
            return super().solve(req, data, stream, reserve)

    reqs = [serve.Request(i, 0.0, "uniform", 100, 1e-4, i) for i in range(70)]  # more than the queue holds
    srv = Server(serve.Tuner(errors=SYNTH), workers=8, hbm_budget=100)
    srv._failed = set()
    t = time.perf_counter()
    res = srv.run(reqs, realtime=False)
    t = time.perf_counter() - t
    assert [r.rid for r in res] == list(range(70)) and all(not r.error for r in res)
    # 64 of them before the first is served, eight at a time
    assert all(64 / 8 * 0.05 <= r.start <= r.done <= t and r.latency == r.done for r in res)
    assert len({i for rid, i in seen if rid < 64}) > 1 and threading.get_ident() not in {i for _, i in seen}
