"""bench.py's BGK leg: enough launches before the clock starts for the part to
settle, whatever --warmup is, on a state that advances by the stated steps alone."""
import pytest
import torch

import bench
from paper_2504_14494_amd import lbm


@pytest.mark.parametrize("warmup,steps", [(5, 20), (50, 1000), (0, 1)])
def test_the_part_settles_before_the_timed_steps(monkeypatch, warmup, steps):
    log = []

    class Lattice:
        def __init__(self, nx, ny):
            self.a, self.b, self.most = "a", "b", lbm.lbm_steps_max(nx, ny)

        def init(self, *fields):
            return self

        def step_bgk(self, tau, n):
            log.extend(["launch"] * -(-n // self.most))
            log.append(n)

        def moments(self, spec):
            return None, None, None, torch.ones(8, dtype=torch.float64)

    class Event:
        def __init__(self, enable_timing):
            pass

        def record(self):
            log.append("event")

        def elapsed_time(self, other):
            return 1.0

    def settle(src, dst, *args):
        assert (src, dst) == ("a", "b")
        log.append("launch")

    monkeypatch.setattr(lbm, "Lattice", Lattice)
    monkeypatch.setattr(lbm, "lbm_steps_bgk", settle)
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    bench.bgk_leg(1024, 1000.0, 0.04, steps, warmup)
    first = log.index("event")
    assert log[:first].count("launch") >= 30
    assert [x for x in log if isinstance(x, int)] == [warmup, steps]
    timed = log[first + 1:log.index("event", first + 1)]
    assert [x for x in timed if isinstance(x, int)] == [steps]
