"""Two steps per launch of lattices periodic along z whose state is larger than 2 GiB, so that the byte offsets
across the lattice exceed 31 bits, against the same steps one by one: equal bit for bit."""
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

BB, FS, PER = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP, L.LBM_BC_PERIODIC


@pytest.mark.parametrize("flags", [0, L.LBM_FLAG_PLAIN_SOA], ids=["planes", "plain"])
@pytest.mark.parametrize("bc", [(PER,) * 6, (BB, FS, BB, BB, PER, PER)], ids=["periodic", "walls"])
@pytest.mark.parametrize("precision,shape", [("f32", (64, 66, 12500)), ("f64", (64, 66, 6250)), ("f64", (1536, 1536, 11))])
def test_offsets_beyond_31_bits(precision, shape, bc, flags):
    sims = []
    for steps in ((1,) * 4, (4,)):
        sim = S.Simulation(shape, 1.6, precision=precision, bc=bc, flags=flags)
        assert (1 << 31) < sim.pops[0].numel() * sim.pops[0].element_size() < (1 << 32)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1710)
        sim.pops[0].uniform_(-0.005, 0.005, generator=gen)
        for n in steps:
            sim.liquid_steps(n)
        sims.append(sim)
    torch.cuda.synchronize()
    a, b = sims
    now = [s.pops[0] if s.pops[0].data_ptr() == L.lbm_state_buffer(s.ctx) else s.pops[1] for s in sims]
    assert torch.isfinite(now[0]).all()
    assert torch.equal(*now)
    a.close()
    b.close()
