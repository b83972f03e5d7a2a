"""The method-step tuning against a stand-in for the library whose steps take known times: what it keeps must
follow from launches its knobs apply to."""
import pytest
import torch

from paper_1710_07073_amd import autotune
from paper_1710_07073_amd import lbm as L


class _Clock:
    """lbm_* calls that only advance a clock: pairs of steps take the same time whatever the cap, but for
    noise; single steps are fastest at one cap."""

    def __init__(self, pair_us, best_cap):
        self.us, self.cap, self.overlap = 0.0, 0, True
        self.pair_us, self.best_cap, self.noise = pair_us, best_cap, 0

    def lbm_get_overlap(self, ctx):
        return True, True

    def lbm_set_overlap(self, ctx, on):
        self.overlap = bool(on)

    def lbm_set_step_occupancy(self, ctx, cap):
        self.cap = cap

    def lbm_run(self, ctx, params, soa, nb, n, graph):
        single = 200.0 + 10.0 * abs(self.cap - self.best_cap) + (0.0 if self.overlap else 25.0)
        self.us += n % 2 * single
        if n >= 2:
            self.noise = (self.noise * 29 + 7) % 31
            self.us += n // 2 * 2 * (self.pair_us[self.overlap] + 0.05 * self.noise)


@pytest.mark.parametrize("best_cap", [0, 4, 7])
@pytest.mark.parametrize("pairs", [{True: 135.0, False: 150.0}, {True: 180.0, False: 150.0}])
def test_method_tuning_keeps_the_cap_of_single_steps(monkeypatch, pairs, best_cap):
    clock = _Clock(pairs, best_cap)
    for name in ("lbm_get_overlap", "lbm_set_overlap", "lbm_set_step_occupancy", "lbm_run"):
        monkeypatch.setattr(L, name, getattr(clock, name))

    class Event:
        def __init__(self, enable_timing):
            pass

        def record(self, stream):
            self.at = clock.us

        def synchronize(self):
            pass

        def elapsed_time(self, other):
            return (other.at - self.at) * 1e-3

    monkeypatch.setattr(torch.cuda, "Event", Event)

    class Sim:
        ctx = stream = params = None

        class bubbles:
            soa, nb = None, 1

    cap, sweep, _ = autotune.tune_method_occupancy(Sim)
    assert (cap, clock.cap) == (best_cap, best_cap)
    assert clock.overlap == (pairs[True] < pairs[False])
