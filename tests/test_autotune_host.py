"""The autotuner's candidates on the CPU: a batch whose members all scan through
record runs launches no direct scan, so its tile and workgroups are not swept."""
from types import SimpleNamespace

import pytest


@pytest.mark.parametrize("runs,count", [((100, 7), 3), ((100, 0), 27), ((0,), 27)])
def test_only_candidates_that_differ(runs, count, monkeypatch):
    from paper_1810_13132_amd import autotune
    batch = SimpleNamespace(sketches=[SimpleNamespace(scan_route=lambda n, r=r: SimpleNamespace(run_records=r)) for r in runs],
                            set_tuning=lambda *a: None)
    monkeypatch.setattr(autotune, "time_steps", lambda b, p, h, o, reps: 1.0)
    best, timings = autotune.tune(batch, [], [], [])
    assert len(timings) == count and {int(k.split(",")[1]) for k in timings} == {16, 64, 256}
    assert best["est_tile"] in (16, 64, 256)
    _, timings = autotune.tune(batch, [], [], [], candidates=[(2048, 16, 4)])
    assert list(timings) == ["2048,16,4"]
