"""One bubble half at velocities whose squares overflow, or nearly, or underflow, against the host's evaluation of
the same closures, on the path that updates a bubble in its interpolation workgroup and on the one with an update
kernel of its own."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

# as for the ordinary range (test_gpu_bubble_update.py): rounding of 11 force evaluations, far inside
TOL = 1e-11


@pytest.mark.parametrize("nb", [1, 300])
@pytest.mark.parametrize("v", [(1e160, 0, 0), (0, -3e200, 0), (1e155, 1e155, -1e155), (1e308, 1e308, 0), (0, 0, 1.5e154),
                               (1e150, 0, 0), (1e120, 1, 0), (1e-160, 2e-160, 0), (0, 0, 1e-170)])
def test_extreme_velocities(v, nb):
    """Finite or not as on the host, and a bubble whose position is lost is reported by the next half."""
    shape, x0 = (32, 32, 64), np.array([10.0, 11.0, 12.0])
    params = S.bubble_params(g=1e-5, sigma=1e-4)
    want = L.host_bubble_ode(params, 0.1, 3.0, x0, np.array(v, float), *np.zeros((3, 3)), shape)
    sim = S.Simulation(shape, 1.25, precision="f64")  # nu = 0.1
    vel = np.zeros((3, nb))
    vel[:, 0] = v
    sim.add_bubbles(np.repeat(x0[:, None], nb, 1), np.full(nb, 3.0), params, vel=vel)
    torch.cuda.synchronize()
    L.bubbles_step(sim.ctx, sim.params, sim.bubbles.soa, nb)
    torch.cuda.synchronize()
    b = sim.bubbles
    for got, w in zip((b.positions(), b.velocities(), b.reactions()), want):
        np.testing.assert_allclose(got[:, 0], w, rtol=TOL, atol=1e-300)
    sim.check()
    if not np.isfinite(want[0]).all():
        L.lbm_step(sim.ctx, 1)
        L.bubbles_step(sim.ctx, sim.params, b.soa, nb)
        with pytest.raises(L.LbmError) as e:
            sim.check()
        assert e.value.code == L.LBM_EINVAL
    sim.close()
