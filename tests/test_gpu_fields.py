"""Density, velocity, sums and populations of a lattice with every face rule against the oracle's
streaming step: the populations are copies (the same bits), the fields are its sums in 64 bits rounded
once, so within two units in the last place; the global sums within N 19 eps."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

BB, FS, PER = O.BC_BOUNCE_BACK, O.BC_FREE_SLIP, O.BC_PERIODIC
C, _, _ = O.lattice()


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [(BB,) * 6, (BB,) * 5 + (FS,), (FS, BB, BB, FS, FS, BB), (PER, PER, BB, FS, BB, BB)],
                         ids=["walls", "top", "mixed", "periodic"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 2), (64, 8, 9), (101, 67, 41), (128, 96, 151)])
def test_fields_match_streaming_by_hand(shape, bc, precision):
    nx, ny, nz = shape
    sim = S.Simulation(shape, 1.3, precision=precision, bc=bc)
    rng = np.random.default_rng(7)
    post = (0.01 * rng.standard_normal((19, nz, ny, nx))).astype(np.float32 if precision == "f32" else np.float64)
    p = L.lbm_state_buffer(sim.ctx)
    buf = sim.pops[0] if sim.pops[0].data_ptr() == p else sim.pops[1]
    buf.view(-1).copy_(torch.as_tensor(np.ascontiguousarray(post.transpose(1, 0, 2, 3)).reshape(-1)))
    g = O.stream(post.astype(np.float64), bc)
    assert np.array_equal(sim.populations().double().cpu().numpy(), g)
    rho, u, sums = sim.moments()
    eps = np.finfo(post.dtype).eps
    r = 1.0 + g.sum(0)
    assert np.abs(rho.double().cpu().numpy() / r - 1.0).max() <= 2 * eps
    m = np.tensordot(np.asarray(C, np.float64).T, g, 1)
    # a velocity's sum of 10 terms of 0.05 at most, in another order
    assert np.abs(u.double().cpu().numpy() - m / r).max() <= 2 * eps * np.abs(m / r).max() + 10 * 0.05 * 2.3e-16
    want = np.array([r.sum(), *m.reshape(3, -1).sum(1)])
    assert np.abs(np.asarray(sums) - want).max() <= r.size * 19 * 2.3e-16
    sim.close()
