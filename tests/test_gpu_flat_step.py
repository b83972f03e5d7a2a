"""The liquid step with a thread per cell in flat order (rows that do not fill the workgroups) against the
same step in workgroups of rows and against a batch of one column: the same bits."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

BB, FS, PER = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP, L.LBM_BC_PERIODIC
WALLS, TOP = (BB,) * 6, (BB,) * 5 + (FS,)


def _bubbles(shape, nb=6):
    rng = np.random.default_rng(9)
    return rng.uniform(0.05, 0.95, (3, nb)) * (np.array(shape)[:, None] - 1), rng.uniform(1.0, 3.0, nb)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [WALLS, TOP, (BB, FS, PER, PER, BB, BB)], ids=["walls", "top", "periodic"])
@pytest.mark.parametrize("overlap", [False, True])
def test_flat_steps_equal_rows(overlap, bc, precision):
    shape = (96, 35, 41)  # rows of 32 threads fill, of 64 do not; 2^17 cells and a part of a workgroup
    pos, d = _bubbles(shape)
    sims = []
    for bx in (32, 64):
        sim = S.Simulation(shape, 1.5, precision=precision, bc=bc)
        sim.add_bubbles(pos, d, S.bubble_params(g=2e-5, sigma=3e-4))
        L.lbm_set_launch(sim.ctx, 1, bx)
        L.lbm_set_overlap(sim.ctx, overlap)
        sim.step(6)
        sim.check()
        sims.append(sim)
    assert torch.equal(sims[0].populations(), sims[1].populations())
    assert torch.equal(sims[0].vel, sims[1].vel)
    assert np.array_equal(sims[0].bubbles.positions(), sims[1].bubbles.positions())


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [WALLS, TOP], ids=["walls", "top"])
@pytest.mark.parametrize("shape", [(67, 50, 41), (1, 400, 331), (65, 1, 2017), (130, 64, 16)])
def test_flat_steps_equal_a_batch_of_one(shape, bc, precision):
    pos, d = _bubbles(shape)
    params = S.bubble_params(g=2e-5, sigma=3e-4)
    sim = S.Simulation(shape, 1.5, precision=precision, bc=bc)
    sim.add_bubbles(pos, d, params)
    batch = S.Batch([dict(shape=shape, omega=1.5, bc=bc, pos=pos, d=d)], params, precision=precision)
    sim.step(5)
    batch.step(5)
    sim.check()
    batch.check()
    assert torch.equal(sim.populations(), batch.populations(0))
    assert np.array_equal(sim.bubbles.positions(), batch.bubbles.positions())
