"""One bubble half against the oracle over the range of the closures' arguments (Re from 1e-9 to 1e3,
every lift branch, every reaction), on the path that updates a bubble in its interpolation workgroup
and on the one with an update kernel of its own; and the force gather of a lattice of few tiles
against the batch's, which takes a wavefront per tile."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

# 11 force evaluations, each within about 16 ulp (2e-15), through sub-steps that do not amplify
# (dt_b times the relaxation rate stays below 2): 4e-14; the slip velocity is a difference of numbers
# up to some ten times its size, and both sides round: 1e-11 of the vector's length holds a margin
TOL = 1e-11


@pytest.mark.parametrize("coupling", [0, O.REACTION_SUBSTEP_MEAN, O.REACTION_NET_FORCE])
@pytest.mark.parametrize("omega,eo", [(1.0, 0.5), (1.98, 2.148), (1.98, 5.0), (1.9, 40.0)])
@pytest.mark.parametrize("nb", [1, 3, 120, 300])
def test_bubble_update_over_reynolds_numbers(nb, omega, eo, coupling):
    shape = (24, 20, 28)
    rng = np.random.default_rng(nb)
    d = rng.uniform(1.5, 3.0, nb)
    pos = np.stack([rng.uniform(0, n - 1, nb) for n in shape])
    speed = 10.0 ** rng.uniform(-9, np.log10(0.3), nb)
    way = rng.normal(size=(3, nb))
    vel = speed * way / np.linalg.norm(way, axis=0)
    g = 1e-5
    kw = dict(g=g, sigma=(1 - 1e-3) * g * 2.2 ** 2 / eo, coupling=coupling)
    U = rng.uniform(-1e-4, 1e-4, (3,) + shape[::-1])
    sim = S.Simulation(shape, omega, precision="f64")
    sim.add_bubbles(pos, d, S.bubble_params(**kw), vel=vel)
    torch.cuda.synchronize()
    sim.vel.copy_(torch.from_numpy(U))
    lat = O.Lattice(*shape, omega)
    lat.U[:] = U
    bub = O.Bubbles(pos=pos.copy(), d=d.copy(), vel=vel.copy())
    psi = O.method_step(lat, O.bubble_params(**kw), bub)
    L.bubbles_step(sim.ctx, sim.params, sim.bubbles.soa, nb)
    torch.cuda.synchronize()
    for got, want in ((sim.bubbles.velocities(), bub.vel), (sim.bubbles.reactions(), psi),
                      (sim.bubbles.positions(), bub.pos)):
        size = np.linalg.norm(want, axis=0)
        assert np.isfinite(got).all()
        assert (np.abs(got - want) <= TOL * size + 1e-300).all(), (np.abs(got - want) / size).max()
    sim.close()


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("shape,nb,d,bc", [
    ((30, 30, 90), 384, 2.5, (0, 0, 0, 0, 0, 1)),   # crowded, some lists overflow
    ((16, 16, 48), 700, 2.0, (0,) * 6),             # every list overflows
    ((24, 20, 33), 40, 3.0, (1, 0, 0, 1, 1, 0)),    # lists only, ragged tiles
    ((33, 17, 25), 200, 2.0, (2, 2, 2, 2, 0, 0)),   # periodic windows
    ((9, 9, 9), 300, 1.0, (2,) * 6),                # windows that wrap onto themselves
    ((64, 64, 128), 65, 2.0, (0,) * 6),             # as many tiles as the workgroup gather takes
    ((64, 64, 129), 65, 2.0, (0,) * 6)])            # one layer of tiles more
def test_gather_by_workgroup_equals_gather_by_wavefront(shape, nb, d, bc, precision):
    rng = np.random.default_rng(1710)
    pos = np.stack([rng.uniform(0, n - 1, nb) for n in shape])
    dd = d * rng.uniform(0.7, 1.2, nb)
    par = S.bubble_params(g=1e-5, sigma=1e-4)
    sim = S.Simulation(shape, 1.5, precision=precision, bc=bc)
    sim.add_bubbles(pos, dd, par)
    batch = S.Batch([dict(shape=shape, omega=1.5, bc=bc, pos=pos, d=dd)], par, precision=precision)
    sim.step(4)
    batch.step(4)
    sim.check()
    batch.check()
    assert sim.populations().abs().max() > 0
    assert torch.equal(sim.populations(), batch.populations(0))
    for k in ("x", "uz", "psiz", "state"):
        assert torch.equal(sim.bubbles.t[k], batch.bubbles.t[k])
    sim.close()
    batch.close()
