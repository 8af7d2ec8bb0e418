"""Admission by the smaller workspace where the full one does not fit, on the CPU with a fake executor."""

import threading
import time

import pytest

from paper_1103_6031_amd.serve import Request, Server


class FakeExec:
    def __init__(self):
        self.lock, self.running, self.most, self.plain = threading.Lock(), 0, 0, {}

    def __call__(self, req, slot):
        with self.lock:
            self.running += 1
            self.most = max(self.most, self.running)
            self.plain[req.id] = req.plain
        time.sleep(0.03)
        with self.lock:
            self.running -= 1
        return 0


def _run(budget, count, full=8, plain=5):
    ex = FakeExec()
    srv = Server(ex, lambda r: full, slots=4, budget_bytes=budget, plain_footprint=lambda r: plain)
    recs = srv.run([Request(i, 0.0, 32) for i in range(count)])
    assert all(r.error is None for r in recs.values()) and srv.peak_bytes <= budget
    return ex, recs


def test_full_workspaces_where_they_fit():
    ex, recs = _run(32, 4)
    assert ex.most == 4 and not any(ex.plain.values())
    assert all(r.footprint == 8 for r in recs.values())


def test_plain_workspaces_where_only_they_fit():
    # 8 + 8 + 5 of 21: the third request runs in its smaller workspace instead of waiting
    ex, recs = _run(21, 3)
    assert ex.most == 3 and ex.plain == {0: False, 1: False, 2: True}
    assert [recs[i].footprint for i in range(3)] == [8, 8, 5]
    assert not any(r.waited_for_memory for r in recs.values())


def test_a_budget_below_the_full_workspace_still_serves():
    ex, recs = _run(5, 2)
    assert ex.most == 1 and all(ex.plain.values())
    with pytest.raises(ValueError):
        _run(4, 1)


def test_footprints_of_real_requests():
    from paper_1103_6031_amd import serve
    r = Request(0, 0.0, 64, [((64,) * 3, (16,) * 3), ((32,) * 3, (16,) * 3)], 2)
    for prec in ("mixed", "fp64"):
        assert 0 < serve.footprint_bytes(r, prec, plain=True) < serve.footprint_bytes(r, prec)
