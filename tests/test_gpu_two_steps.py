"""Two liquid steps per launch against the same steps one by one: the arithmetic of a cell and its
order are the same, so every field is equal bit for bit. Sizes at the edges of the pass: whole rows
and pieces of rows, one and many tiles and chunks, remainders, slabs at the walls and over the whole
lattice."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

BB, FS, PER = 0, 1, 2
WALLS = (BB,) * 6
TOP = (BB, BB, BB, BB, BB, FS)
MIXED = (FS, BB, BB, FS, FS, BB)
SLIP = (FS,) * 6
ARRAYS = ("x", "y", "z", "ux", "uy", "uz", "ulx", "uly", "ulz", "state", "psix", "psiy", "psiz")


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


def _state(sim):
    p = L.lbm_state_buffer(sim.ctx)
    return sim.pops[0] if sim.pops[0].data_ptr() == p else sim.pops[1]


def _same(a, b):
    torch.cuda.synchronize()
    assert torch.isfinite(_state(a)).all()
    assert torch.equal(_state(a), _state(b))
    assert torch.equal(a.vel, b.vel)
    assert torch.equal(a.force, b.force)
    if a.bubbles is not None:
        for k in ARRAYS:
            assert torch.equal(a.bubbles.t[k], b.bubbles.t[k]), k
    a.close()
    b.close()


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [WALLS, TOP, MIXED, SLIP, (PER,) * 6, (BB, BB, PER, PER, PER, PER),
                                (PER, PER, BB, BB, BB, FS), (BB, FS, BB, BB, PER, PER)],
                         ids=lambda b: "".join(map(str, b)))
def test_liquid_pairs_equal_single_steps(bc, precision):
    """Liquid alone: even and odd step counts, every face kind, rows that fill a workgroup, that
    leave threads idle, that are cut in pieces with and without a remainder; thin lattices."""
    # FP64 takes pairs from 2^17 cells on, FP32 from 9 2^16 on
    for shape in ([(128, 64, 17), (37, 61, 60), (300, 45, 10), (1100, 40, 3), (31, 2200, 2), (129, 33, 40)]
                  if precision == "f64" else
                  [(128, 64, 73), (37, 61, 263), (300, 45, 44), (1100, 40, 14), (31, 2200, 9), (129, 33, 139)]):
        a, b = _sim(shape, precision, bc), _sim(shape, precision, bc)
        for _ in range(5):
            a.liquid_steps(1)
        b.liquid_steps(5)
        _same(a, b)


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [TOP, (BB, BB, PER, PER, PER, PER)], ids=["walls", "periodic"])
@pytest.mark.parametrize("flags", [L.LBM_FLAG_STATIC_FORCE, L.LBM_FLAG_WRITE_U_ALL,
                                   L.LBM_FLAG_PLAIN_SOA,
                                   L.LBM_FLAG_WRITE_U_ALL | L.LBM_FLAG_PLAIN_SOA])
def test_liquid_pairs_with_flags(flags, bc, precision):
    """A static force field, the velocity written everywhere, the plain layout."""
    a, b = (_sim((96, 71, 33 if precision == "f64" else 88), precision, bc, flags) for _ in range(2))
    for _ in range(4):
        a.liquid_steps(1)
    b.liquid_steps(4)
    _same(a, b)


def _bubbles(shape, nb, d, seed, z):
    rng = np.random.default_rng(seed)
    return (np.stack([rng.uniform(0, shape[0] - 1, nb), rng.uniform(0, shape[1] - 1, nb),
                      rng.uniform(z[0] * (shape[2] - 1), z[1] * (shape[2] - 1), nb)]),
            d * rng.uniform(0.8, 1.2, nb), rng.uniform(-1, 1, nb))


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [WALLS, TOP, MIXED], ids=["walls", "top", "mixed"])
@pytest.mark.parametrize("nb,d,z", [(1, 3.0, (0.3, 0.5)), (1, 2.0, (0.0, 0.02)), (1, 2.0, (0.97, 0.99)),
                                    (7, 2.5, (0.0, 0.3)), (7, 0.7, (0.0, 1.0)), (300, 2.0, (0.4, 0.9))])
def test_method_step_pairs_equal_single_steps(nb, d, z, bc, precision):
    """With bubbles, through lbm_run eagerly and in graphs (4 and 10 steps), then liquid alone over the
    flagged tiles the last bubble half left."""
    shape = (96, 80, 70 if precision == "f64" else 104)  # 3 2^17 cells and 3 2^18
    pos, dd, _ = _bubbles(shape, nb, d, 3, z)
    for steps, graph in ((7, 0), (12, 4), (21, 10)):
        stream = torch.cuda.Stream()
        sims = []
        for paired in (False, True):
            torch.cuda.synchronize()
            sim = _sim(shape, precision, bc, stream=stream)
            sim.add_bubbles(pos, dd, S.bubble_params(g=1e-4, sigma=1e-3))
            torch.cuda.synchronize()
            if paired:
                sim.run(steps, graph_steps=graph)
                sim.liquid_steps(3)
            else:
                sim.step(steps)
                for _ in range(3):
                    sim.liquid_steps(1)
            sim.check()
            sims.append(sim)
        _same(*sims)


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("bc", [WALLS, TOP, MIXED], ids=["walls", "top", "mixed"])
@pytest.mark.parametrize("nb,d,z", [(1, 3.0, (0.3, 0.5)), (1, 2.0, (0.0, 0.02)), (7, 2.0, (0.0, 1.0)),
                                    (300, 2.0, (0.4, 0.9))])
def test_overlapped_pairs_equal_single_steps(nb, d, z, bc, precision):
    """The same with the bubble kernels and the slab's first step beside the rest of the lattice, single
    overlapped steps in between (odd counts, calls of one step) and bubbles moved from the host."""
    shape = (96, 80, 70 if precision == "f64" else 104)  # 3 2^17 cells and 3 2^18
    pos, dd, _ = _bubbles(shape, nb, d, 3, z)
    for steps, graph in ((8, 0), (12, 4), (31, 10)):
        stream = torch.cuda.Stream()
        sims = []
        for paired in (False, True):
            torch.cuda.synchronize()
            sim = _sim(shape, precision, bc, stream=stream)
            sim.add_bubbles(pos, dd, S.bubble_params(g=1e-4, sigma=1e-3))
            L.lbm_set_overlap(sim.ctx, paired)
            torch.cuda.synchronize()
            for n in (steps, 3):
                if paired:
                    sim.run(n, graph_steps=graph)
                else:
                    sim.step(n)
                with torch.cuda.stream(stream):
                    sim.bubbles.t["z"].copy_(torch.from_numpy(pos[2][::-1].copy()))
            sim.run(1) if paired else sim.step(1)
            sim.check()
            sims.append(sim)
        _same(*sims)


def test_overlapped_pair_reports_a_bubble_beyond_its_slab():
    """A bubble thrown further than the slab's margin is reported, as by an overlapped step."""
    sim = _sim((96, 80, 104), "f32", WALLS)
    sim.add_bubbles([[40.0], [40.0], [20.0]], [2.0], S.bubble_params(g=1e-4, sigma=1e-3),
                    vel=np.array([[0.0], [0.0], [24.0]]))
    L.lbm_set_overlap(sim.ctx, True)
    sim.run(2)
    with pytest.raises(L.LbmError) as e:
        sim.check()
    assert e.value.code == L.LBM_EUNSUPPORTED
    sim.close()


@pytest.mark.parametrize("speed", [0.5, 3.0, 20.0])
@pytest.mark.parametrize("nb", [1, 5, 300])
def test_pairs_follow_fast_bubbles(nb, speed):
    """Bubbles thrown along z, several cells in one step: the planes of a pair follow them."""
    shape = (96, 80, 104)
    pos, dd, v = _bubbles(shape, nb, 2.0, 5, (0.2, 0.8))
    sims = []
    for paired in (False, True):
        sim = _sim(shape, "f32", TOP)
        sim.add_bubbles(pos, dd, S.bubble_params(g=1e-4, sigma=1e-3),
                        vel=np.stack([0 * v, 0 * v, speed * v]))
        torch.cuda.synchronize()
        sim.run(6) if paired else sim.step(6)
        sim.check()
        sims.append(sim)
    _same(*sims)
