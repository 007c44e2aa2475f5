"""The 3D passes and front at the edges of their column tiles and z chunks."""
import copy

import numpy as np
import pytest

from paper_1907_13088_amd import inputs as I

from gpu_helpers import log, rel_err, run_gpu, run_oracle
from test_gpu_3d import _reshape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def waves():
    return {dt: I.planewave_3d(n=132, kidx=2, npulses=4, sigma=3.0, filter_passes=1, tol=0.0, m_max=7, steps=2,
                               seed=3020, dtype=dt) for dt in ("f32", "f64")}


# (nz, ny, nx): a tile writes 62, 60 or 58 columns by 4 to 24 rows (one to
# three sweeps per pass, two sizes of tile), a chunk is of two planes or more;
# each value stands at, just under or just over one of these
@pytest.mark.parametrize("shape", [(2, 12, 58), (3, 13, 59), (2, 20, 60), (5, 21, 61), (4, 6, 62), (7, 7, 63),
                                   (33, 14, 64), (9, 15, 65), (6, 60, 116), (11, 25, 131), (131, 3, 30)])
@pytest.mark.parametrize("dtype,solver", [("f32", 0), ("f32", 1), ("f64", 0), ("f64", 1)])
def test_3d_tile_edges(waves, dtype, solver, shape):
    """Seven sweeps in the deepest passes (with their shorter last one) and in
    passes of one sweep are bitwise equal, and within the FP64 (1e-12) or
    FP32 (1e-5) bound of the oracle."""
    w = _reshape(copy.copy(waves[dtype]), shape)
    Ed, Bd, _, k = run_gpu(w, 2, sweeps=7, tol=0.0, solver=solver)
    E1, B1, _, _ = run_gpu(w, 2, sweeps=7, tol=0.0, spp=1, solver=solver)
    for a, b in zip(Ed + Bd, E1 + B1):
        assert np.array_equal(a, b)
    Eo, Bo, _ = run_oracle(w, 2, sweeps=7, tol=0.0, solver=solver)
    e = rel_err(Ed + Bd, Eo + Bo)
    log(f"3D tile edges {dtype} solver {solver} {shape}, depth {k}: {max(e):.2e}")
    assert max(e) < (1e-12 if dtype == "f64" else 1e-5)
