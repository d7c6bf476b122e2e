"""bench.py's wall-clock timing: calls until the clocks have settled, the warm-up, then
exactly the timed calls between two synchronisations."""
import os
import sys
import time
from types import SimpleNamespace

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def run(steps, warmup, **kw):
    events = []
    torch = SimpleNamespace(cuda=SimpleNamespace(synchronize=lambda: events.append("sync")))

    def fn():
        events.append(time.perf_counter())
        time.sleep(0.001)

    t = bench.timed(fn, steps, warmup, torch, **kw)
    return t, events


def test_timed_calls():
    t, events = run(7, 3)
    assert [e == "sync" for e in events] == [False] * 3 + [True] + [False] * 7 + [True]
    assert 0.001 <= t < 0.1


def test_comparisons_settle_before_they_are_timed():
    _, events = run(4, 2, settle_ms=60.0)
    calls = [e for e in events if e != "sync"]
    timed = events[-5:]
    assert timed[-1] == "sync" and "sync" not in timed[:-1] and events[-6] == "sync"
    assert timed[0] - calls[0] >= 0.06
