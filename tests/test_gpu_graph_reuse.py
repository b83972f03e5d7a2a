"""The graphs lbm_run captures: a call like an earlier one replays them, and one that is replaced outlives its
replay."""
import time

import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("overlap", [0, 1])
@pytest.mark.parametrize("graph", [2, 6, 10])
def test_later_calls_capture_nothing(graph, overlap):
    """Three replays per call, odd numbers of pairs in each. The host time of a call is compared with that of
    calls that must capture again, because the occupancy their launches hold changed."""
    shape = (96, 80, 104)
    stream = torch.cuda.Stream()
    sim = S.Simulation(shape, 1.6, precision="f32", stream=stream)
    rng = np.random.default_rng(1)
    sim.add_bubbles(np.stack([rng.uniform(8, n - 9, 3) for n in shape]), np.full(3, 2.0),
                    S.bubble_params(g=1e-7, sigma=1e-4))
    L.lbm_set_overlap(sim.ctx, overlap)
    torch.cuda.synchronize()

    def call():
        t0 = time.perf_counter()
        sim.run(3 * graph, graph_steps=graph)
        t = time.perf_counter() - t0
        stream.synchronize()
        return t

    for _ in range(3):
        call()
    again = min(call() for _ in range(30))
    anew = []
    for k in range(30):
        L.lbm_set_step_occupancy(sim.ctx, 1 + k)
        anew.append(call())
    print(f"[case] graphs of {graph}, overlap {overlap}: {again * 1e6:.0f} us a call, {min(anew) * 1e6:.0f} us with "
          "a capture", flush=True)
    assert again < 0.75 * min(anew)
    sim.close()


def test_graphs_replaced_while_they_replay():
    """Captures follow each other faster than their replays end, and the context goes away during the last: a
    replaced graph outlives its replay, and the steps are those of a run without graphs."""
    shape = (96, 80, 104)
    stream = torch.cuda.Stream()
    sims = []
    for graphs in (True, False):
        sim = S.Simulation(shape, 1.6, precision="f32", stream=stream)
        rng = np.random.default_rng(1)
        sim.add_bubbles(np.stack([rng.uniform(8, n - 9, 3) for n in shape]), np.full(3, 2.0),
                        S.bubble_params(g=1e-5, sigma=1e-4))
        L.lbm_set_overlap(sim.ctx, 1)
        torch.cuda.synchronize()
        for k in range(30):
            L.lbm_set_step_occupancy(sim.ctx, 1 + k)
            sim.run(6, graph_steps=2 if graphs else 0)
        pops = sim.pops[0] if sim.pops[0].data_ptr() == L.lbm_state_buffer(sim.ctx) else sim.pops[1]
        if not graphs:
            sim.check()
        sims.append((sim, pops))
        sim.close()  # the buffers stay
        stream.synchronize()
    (a, p), (b, q) = sims
    assert torch.isfinite(p).all() and torch.equal(p, q)
    for k in ("x", "y", "z", "ux", "uy", "uz"):
        assert torch.equal(a.bubbles.t[k], b.bubbles.t[k]), k
