"""A caller that binds buffers of its own, or replays graphs of its own that name them, finds the state of n
steps in the buffer that n single steps leave it in, however many of them a launch takes."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

pytestmark = pytest.mark.gpu

BB, FS, PER = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP, L.LBM_BC_PERIODIC
TOP = (BB,) * 5 + (FS,)
CHANNEL = (BB, BB, PER, PER, PER, PER)
SHAPE = (96, 80, 104)  # 3 2^18 FP32 cells: with walls, liquid and method steps go in pairs
PARAMS = dict(g=1e-4, sigma=1e-3)


def _sim(bc, stream, nb, overlap=0):
    sim = S.Simulation(SHAPE, 1.6, precision="f32", bc=bc, stream=stream)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1710)
    torch.cuda.synchronize()
    for t in (sim.pops[0], sim.vel):
        t.copy_((torch.rand(t.shape, generator=gen, device="cuda") - 0.5) * 0.01)
    rng = np.random.default_rng(7)
    sim.add_bubbles(np.stack([rng.uniform(8, n - 9, nb) for n in SHAPE]), np.full(nb, 2.0), S.bubble_params(**PARAMS))
    L.lbm_set_overlap(sim.ctx, overlap)
    torch.cuda.synchronize()
    return sim


def _advance(sim, how, n):
    if how == "step":
        L.lbm_step(sim.ctx, n)
    else:
        L.lbm_run(sim.ctx, sim.params, sim.bubbles.soa, sim.bubbles.nb, n, 0)


def _same(a, b):
    torch.cuda.synchronize()
    for x, y in ((a.pops[0], b.pops[0]), (a.vel, b.vel), (a.force, b.force), (a.bubbles.t["z"], b.bubbles.t["z"])):
        assert torch.isfinite(x).all()
        assert torch.equal(x, y)


CASES = [("step", TOP, 0, 0), ("step", CHANNEL, 0, 0), ("run", TOP, 0, 0), ("run", TOP, 3, 0), ("run", TOP, 3, 1)]


@pytest.mark.parametrize("n", [2, 4, 6])
@pytest.mark.parametrize("how,bc,nb,overlap", CASES)
def test_callers_graph_of_steps_replays(how, bc, nb, overlap, n):
    stream = torch.cuda.Stream()
    a, b = _sim(bc, stream, nb, overlap), _sim(bc, stream, nb)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        _advance(a, how, n)
    with torch.cuda.stream(stream):
        for k in range(5):
            graph.replay()
            stream.synchronize()
            _advance(a, how, 2 * k)  # eager steps between the replays
    for _ in range(5 * n + 20):
        _advance(b, how, 1)
    a.check()
    _same(a, b)


@pytest.mark.parametrize("how,bc,nb,overlap", CASES)
def test_bound_buffers_receive_the_steps(how, bc, nb, overlap):
    """Every number of steps from a bound state buffer ends in the buffer its parity says."""
    stream = torch.cuda.Stream()
    a, b = _sim(bc, stream, nb, overlap), _sim(bc, stream, nb)
    own = [a.pops[0].clone(), torch.empty_like(a.pops[0])]
    torch.cuda.synchronize()
    L.lbm_bind_buffers(a.ctx, own[0].data_ptr(), own[1].data_ptr(), None)
    at = 0
    for n in (2, 1, 3, 4, 5, 6, 7, 10, 13):
        _advance(a, how, n)
        for _ in range(n):
            _advance(b, how, 1)
        at ^= n & 1
        torch.cuda.synchronize()
        a.check()
        assert L.lbm_state_buffer(a.ctx) == own[at].data_ptr(), n
        assert torch.equal(own[at], b.pops[at]), n
    L.lbm_bind_buffers(a.ctx, a.pops[0].data_ptr(), a.pops[1].data_ptr(), None)


def _batch(stream):
    rng = np.random.default_rng(3)
    cols = [dict(shape=s, omega=1.5, bc=TOP, pos=rng.uniform(0.3, 0.7, (3, nb)) * (np.array(s)[:, None] - 1),
                 d=np.full(nb, 2.0)) for s, nb in (((96, 92, 110), 3), ((57, 31, 60), 0), ((33, 30, 31), 1))]
    batch = S.Batch(cols, S.bubble_params(**PARAMS), precision="f32", stream=stream)  # more than 2^20 cells
    torch.cuda.synchronize()
    return batch


def _columns(batch):
    torch.cuda.synchronize()
    batch.check()
    out = [batch.populations(c) for c in range(batch.ncols)] + [torch.as_tensor(batch.bubbles.positions())]
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n", [2, 4, 6])
def test_callers_graph_of_batch_steps_replays(n):
    stream = torch.cuda.Stream()
    a, b = _batch(stream), _batch(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(n)
    with torch.cuda.stream(stream):
        for k in range(5):
            graph.replay()
            stream.synchronize()
            a.step(2 * k)  # eager steps between the replays
    for _ in range(5 * n + 20):
        b.step(1)
    for x, y in zip(_columns(a), _columns(b)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("what", ["populations", "moments", "checkpoint", "state buffer"])
def test_callers_graph_that_reads_the_state(what):
    """A captured export shows the state after any even number of steps, as it does after single ones."""
    stream = torch.cuda.Stream()
    a = _sim(TOP, stream, 3)
    out = [torch.zeros_like(a.pops[0]), torch.zeros_like(a.vel)]
    torch.cuda.synchronize()

    def export():
        if what == "populations":
            L.lbm_populations(a.ctx, out[0].data_ptr())
        elif what == "moments":
            L.moments(a.ctx, None, out[1].data_ptr(), False)
        elif what == "checkpoint":
            L.lbm_checkpoint(a.ctx, out[0].data_ptr(), out[1].data_ptr())
        else:
            out[0].copy_(a.pops[0] if L.lbm_state_buffer(a.ctx) == a.pops[0].data_ptr() else a.pops[1])

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        export()
    with torch.cuda.stream(stream):
        for n in (2, 4, 6, 2):
            _advance(a, "run", n)
            graph.replay()
            stream.synchronize()
            got = [t.clone() for t in out]
            export()
            stream.synchronize()
            assert torch.isfinite(got[0]).all() and any(t.abs().max() > 0 for t in got)
            assert all(torch.equal(x, y) for x, y in zip(got, out)), n
