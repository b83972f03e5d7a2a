"""A batch of 2^20 cells or more takes its method steps in pairs, two liquid steps per launch: the same
bits as steps one at a time, in every column, eager and replayed."""
import numpy as np
import pytest
import torch

from paper_1710_07073_amd import lbm as L
from paper_1710_07073_amd import sim as S

BB, FS = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP
PARAMS = dict(g=2e-5, sigma=3e-4)


def _columns(top, seed=5):
    # one tile and several, ragged rows and whole lines, a column without bubbles, the smallest; bubbles at
    # the bottom, spread over the height, and at the top
    rng = np.random.default_rng(seed)
    out = []
    for shape, nb, z in (((96, 92, 110), 3, (0.0, 0.1)), ((57, 31, 60), 1, (0.4, 0.5)), ((64, 24, 48), 8, (0.0, 1.0)),
                         ((24, 46, 40), 0, (0, 1)), ((1, 3, 2), 0, (0, 1)), ((33, 30, 31), 2, (0.9, 1.0))):
        ext = np.array(shape)
        pos = rng.uniform(0.2, 0.8, (3, nb)) * (ext[:, None] - 1)
        pos[2] = rng.uniform(*z, nb) * (shape[2] - 1)
        out.append(dict(shape=shape, omega=float(rng.uniform(0.8, 1.8)), bc=(BB,) * 5 + (top,), pos=pos,
                        d=rng.uniform(1.0, 3.5, nb), vel=rng.uniform(-0.05, 0.05, (3, nb))))
    return out


def _batch(cols, precision, stream=None):
    b = S.Batch(cols, S.bubble_params(**PARAMS), precision=precision, stream=stream)
    torch.cuda.synchronize()
    return b


def _state(b, ncols):
    b.check()
    out = [b.populations(c) for c in range(ncols)] + [torch.as_tensor(b.bubbles.positions())]
    torch.cuda.synchronize()  # the batch writes them on its own stream
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("top", [BB, FS])
def test_batch_pairs_equal_single_steps(top, precision):
    cols = _columns(top)
    one, two = _batch(cols, precision), _batch(cols, precision)
    for n in (2, 5, 8):
        for _ in range(n):
            one.step(1)
        two.step(n)
        for a, b in zip(_state(one, len(cols)), _state(two, len(cols))):
            assert torch.equal(a, b), n


@pytest.mark.gpu
@pytest.mark.parametrize("graph", [2, 4, 6, 10])
def test_batch_pairs_replayed(graph):
    cols = _columns(FS)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    one, two = _batch(cols, "f32"), _batch(cols, "f32", stream=stream)
    for n in (graph, 3 * graph + 3):
        for _ in range(n):
            one.step(1)
        two.run(n, graph)
        stream.synchronize()
        for a, b in zip(_state(one, len(cols)), _state(two, len(cols))):
            assert torch.equal(a, b), n
