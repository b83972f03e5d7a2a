"""The tile mask and the force of its flagged tiles in one launch, against the mask's own copy and the
force field: the same values in flagged tiles, the destination untouched elsewhere
(everywhere the same values where a face is not bounce-back, whose adjoint reads every cell)."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import adjoint as A
from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("top", [L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP])
@pytest.mark.parametrize("shape", [(24, 24, 40), (29, 9, 37), (7, 7, 7)])
def test_step_inputs_copy_the_flagged_tiles(shape, top, precision):
    sim = S.Simulation(shape, 1.4, precision=precision, bc=(0,) * 5 + (top,))
    ext = np.array(shape)
    sim.add_bubbles(np.array([[0.5, 0.1], [0.5, 0.9], [0.3, 0.95]]) * (ext[:, None] - 1), [1.0, 0.7],
                    S.bubble_params(g=1e-4, sigma=1e-3))
    L.bubbles_step(sim.ctx, sim.params, sim.bubbles.soa, 2)
    n = L.lbm_step_tiles(sim.ctx)
    mask, tiles = (torch.full((n,), 7, dtype=torch.uint8, device="cuda") for _ in range(2))
    force = torch.full_like(sim.force, 5.0)
    L.lbm_step_tiles(sim.ctx, A._p(mask))
    L.lbm_step_inputs(sim.ctx, A._p(tiles), A._p(force))
    assert torch.equal(mask, tiles)
    t = [-(-e // 8) for e in shape]
    cells = mask.view(t[2], t[1], t[0]).bool()
    for axis in range(3):
        cells = cells.repeat_interleave(8, axis)
    cells = cells[:shape[2], :shape[1], :shape[0]] | (top != L.LBM_BC_BOUNCE_BACK)
    want = torch.where(cells, sim.force.view(3, *shape[::-1]), torch.full_like(force, 5.0).view(3, *shape[::-1]))
    assert torch.equal(force.view(3, *shape[::-1]), want)
    L.lbm_step(sim.ctx, 1)
    sim.check()
