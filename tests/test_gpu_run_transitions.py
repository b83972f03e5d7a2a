"""lbm_run on one live context whose bubbles and way of stepping change from call to call: pairs of steps
beside the bubbles, without bubbles, with more than an overlapped pair takes, in series. What one call leaves
in the library (the box marked ahead for a next pair) must not show in the next."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

BB, FS = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP
TOP = (BB,) * 5 + (FS,)
ARRAYS = ("x", "y", "z", "ux", "uy", "uz", "ulx", "uly", "ulz", "state", "psix", "psiy", "psiz")


def _state(sim):
    p = L.lbm_state_buffer(sim.ctx)
    return sim.pops[0] if sim.pops[0].data_ptr() == p else sim.pops[1]


def _sim(shape, precision, bc, flags=0, stream=None):
    sim = S.Simulation(shape, 1.6, precision=precision, bc=bc, flags=flags, stream=stream)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1710)

    def rand(t, amp):
        torch.cuda.synchronize()
        t.copy_((torch.rand(t.shape, generator=gen, device="cuda", dtype=sim.dtype) - 0.5) * amp)

    rand(_state(sim), 0.01)
    rand(sim.vel, 0.01)
    if flags & L.LBM_FLAG_STATIC_FORCE:
        rand(sim.force, 1e-4)
    torch.cuda.synchronize()
    return sim


def _bubbles(shape, nb, seed):
    rng = np.random.default_rng(seed)
    pos = np.stack([rng.uniform(0, shape[0] - 1, nb), rng.uniform(0, shape[1] - 1, nb),
                    rng.uniform(0.1, 0.8, nb) * (shape[2] - 1)])
    return pos, 2.0 * rng.uniform(0.8, 1.2, nb)


@pytest.mark.parametrize("graph", [0, 4])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_run_after_a_change_of_bubbles_equals_single_steps(precision, graph):
    """Overlapped pairs, none left, more than run beside the liquid, overlap off, none left again."""
    shape = (96, 80, 70 if precision == "f64" else 104)  # 3 2^17 cells and 3 2^18
    stream = torch.cuda.Stream()
    sims = []
    for paired in (False, True):
        torch.cuda.synchronize()
        sim = _sim(shape, precision, TOP, stream=stream)
        params = S.bubble_params(g=1e-4, sigma=1e-3)
        for overlap, nb, steps in ((1, 5, 8), (1, 0, 8), (1, 0, 3), (1, 300, 6), (0, 5, 4), (1, 5, 2), (0, 0, 5)):
            torch.cuda.synchronize()
            L.lbm_set_overlap(sim.ctx, overlap if paired else 0)
            sim.bubbles = None
            if nb:
                sim.add_bubbles(*_bubbles(shape, nb, nb), params)
            torch.cuda.synchronize()
            if paired:
                sim.run(steps, graph_steps=graph)
            else:
                for _ in range(steps):
                    sim.run(1)
            torch.cuda.synchronize()
            sim.check()
        sims.append(sim)
    a, b = sims
    assert torch.isfinite(_state(a)).all()
    assert torch.equal(_state(a), _state(b))
    assert torch.equal(a.vel, b.vel)
    assert torch.equal(a.force, b.force)
    a.close()
    b.close()
