"""Two liquid steps per launch against the same steps one by one, bit for bit, on FP32 lattices with free-slip faces
of the sizes from which pairs are chosen there (with walls, periodic axes and in FP64 they are from smaller ones,
test_gpu_two_steps.py); and on lattices beside the choice, which take single steps."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

BB, FS = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP
TOP, MIXED, SLIP = (BB,) * 5 + (FS,), (FS, BB, BB, FS, FS, BB), (FS,) * 6
ARRAYS = ("x", "y", "z", "ux", "uy", "uz", "ulx", "uly", "ulz", "state", "psix", "psiy", "psiz")


def _sim(shape, precision, bc, stream=None):
    sim = S.Simulation(shape, 1.6, precision=precision, bc=bc, stream=stream)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1710)
    torch.cuda.synchronize()
    for t in (sim.pops[0], sim.vel):
        t.copy_((torch.rand(t.shape, generator=gen, device="cuda", dtype=sim.dtype) - 0.5) * 0.01)
    torch.cuda.synchronize()
    return sim


def _same(a, b):
    torch.cuda.synchronize()
    p, q = (s.pops[0] if s.pops[0].data_ptr() == L.lbm_state_buffer(s.ctx) else s.pops[1] for s in (a, b))
    assert torch.isfinite(p).all()
    assert torch.equal(p, q) and torch.equal(a.vel, b.vel) and torch.equal(a.force, b.force)
    if a.bubbles is not None:
        for k in ARRAYS:
            assert torch.equal(a.bubbles.t[k], b.bubbles.t[k]), k
    a.close()
    b.close()


@pytest.mark.parametrize("bc", [TOP, MIXED, SLIP], ids=["top", "mixed", "slip"])
@pytest.mark.parametrize("shape", [(128, 100, 100), (101, 67, 251), (300, 45, 113), (1100, 40, 40), (129, 63, 200),
                                   (8, 8, 10000), (16, 16, 2400), (48, 48, 300)])
def test_liquid(shape, bc):
    a, b = _sim(shape, "f32", bc), _sim(shape, "f32", bc)
    for _ in range(5):
        a.liquid_steps(1)
    b.liquid_steps(5)
    _same(a, b)


@pytest.mark.parametrize("bc", [TOP, MIXED], ids=["top", "mixed"])
@pytest.mark.parametrize("shape", [(128, 100, 100), (101, 67, 251)])
@pytest.mark.parametrize("nb,d,z", [(1, 3.0, (0.3, 0.5)), (1, 2.0, (0.0, 0.02)), (7, 2.5, (0.0, 1.0)), (300, 2.0, (0.4, 0.9))])
def test_method_steps(nb, d, z, shape, bc):
    rng = np.random.default_rng(3)
    pos = np.stack([rng.uniform(0, shape[0] - 1, nb), rng.uniform(0, shape[1] - 1, nb),
                    rng.uniform(z[0] * (shape[2] - 1), z[1] * (shape[2] - 1), nb)])
    dd = d * rng.uniform(0.8, 1.2, nb)
    for steps, graph in ((7, 0), (21, 10)):
        stream = torch.cuda.Stream()
        sims = []
        for paired in (False, True):
            sim = _sim(shape, "f32", bc, stream=stream)
            sim.add_bubbles(pos, dd, S.bubble_params(g=1e-4, sigma=1e-3))
            L.lbm_set_overlap(sim.ctx, 0)
            torch.cuda.synchronize()
            sim.run(steps, graph_steps=graph) if paired else sim.step(steps)
            sim.check()
            sims.append(sim)
        _same(*sims)
