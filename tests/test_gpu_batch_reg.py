"""Batches on register tiles: the default schedule of small batches."""
import numpy as np
import pytest

from paper_1907_13088_amd import inputs as I

from gpu_helpers import run_gpu, to_np
from test_gpu_batch import _batch

pytestmark = pytest.mark.gpu

# single cells and rows, tiles met exactly and just exceeded, long thin grids
SHAPES = [(1, 1), (3, 2), (22, 51), (23, 52), (26, 54), (64, 64), (65, 129), (5, 700), (300, 9), (110, 240)]


# the fewest sweeps, one pass and its remainder, many passes; odd counts of
# steps hand B back in the last pass
@pytest.mark.parametrize("m,nsteps", [(1, 1), (2, 3), (7, 2), (13, 3), (41, 1)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_register_batch_equals_row_streams_and_single_grids(dtype, m, nsteps):
    """Bitwise equal to the row-streaming schedule (passes of an explicit
    depth) and to each grid stepped alone by the row streams."""
    import torch
    ws = [I.modes_2d((nx, ny), courant=0.3 + 0.04 * k, nmodes=6, npulses=0, m=m, steps=nsteps, seed=4600 + k,
                     dtype=dtype) for k, (ny, nx) in enumerate(SHAPES)]
    out = {}
    for spp in (0, 3):
        b, fields = _batch(ws, dtype, spp)
        b.step(nsteps)
        torch.cuda.synchronize()
        out[spp] = [to_np(E + B) for E, B in fields]
        b.close()
    for g, w in enumerate(ws):
        Eg, Bg, _, _ = run_gpu(w, nsteps, tol=0.0, sweeps=m, variant=3)
        for a, s, t in zip(out[0][g], out[3][g], Eg + Bg):
            assert np.array_equal(a, s) and np.array_equal(a, t), (SHAPES[g], m)


def test_register_batch_of_many_grids():
    """More grids than a wavefront has lanes: the workgroups' search for their
    grid goes on beyond the first 64."""
    import torch
    ws = [I.modes_2d((20 + 7 * (k % 13), 9 + 5 * (k % 11)), courant=0.5, nmodes=4, npulses=0, m=5, steps=2,
                     seed=4700 + k, dtype="f64") for k in range(131)]
    out = {}
    for spp in (0, 3):
        b, fields = _batch(ws, "f64", spp)
        b.step(2)
        torch.cuda.synchronize()
        out[spp] = [to_np(E + B) for E, B in fields]
        b.close()
    for g in range(len(ws)):
        for a, s in zip(out[0][g], out[3][g]):
            assert np.array_equal(a, s), g
