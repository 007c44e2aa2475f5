"""3D passes on wide tiles (taken where two more columns per tile save a column
of tiles): the columns beyond a wave's own come from memory, over the periodic
edge, tile edges and remainders, every pass depth and form."""
import numpy as np
import pytest

from paper_1907_13088_amd import inputs as I
from paper_1907_13088_amd import mx

from gpu_helpers import log, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _noise(shape, dtype, tol=0.0, p=1):
    w = I.planewave_3d(n=8, kidx=1, npulses=1, sigma=1.0, filter_passes=p, tol=tol, m_max=300, steps=2, seed=3022, dtype=dtype)
    rng = np.random.default_rng(sum(shape))
    w.shape = shape
    w.E, w.B, w.J0 = ([rng.standard_normal(shape).astype(np.float32).astype(np.float64) for _ in range(3)]
                      for _ in range(3))
    return w


# (nz, ny, nx): a wide tile writes 64, 62 or 60 columns in passes of one, two or
# three sweeps, a narrow one two fewer; the widths stand at and around multiples
SHAPES = [(5, 7, 59), (4, 30, 60), (9, 13, 61), (6, 5, 62), (3, 14, 63), (7, 20, 64), (5, 40, 119), (4, 9, 120), (3, 8, 124),
          (6, 11, 128), (2, 25, 180), (4, 6, 186), (1, 3, 60), (2, 2, 62), (5, 1, 200), (3, 4, 130), (4, 8, 70), (6, 9, 90), (1, 40, 150)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_depths_agree_bitwise_and_match_the_oracle(shape, dtype):
    w = _noise(shape, dtype)   # (one or two planes run single sweeps, few rows the lowest tiles)
    for solver in (mx.SOLVER_ALG1, mx.SOLVER_CHEBYSHEV):
        runs = [run_gpu(w, 2, sweeps=7, tol=0.0, spp=k, solver=solver) for k in ((0, 1, 2) if dtype == "f32" else (0, 1))]
        for r in runs[1:]:
            for a, b in zip(runs[0][0] + runs[0][1], r[0] + r[1]):
                assert np.array_equal(a, b)
        Eo, Bo, _ = run_oracle(w, 2, sweeps=7, tol=0.0, solver=solver)
        e = rel_err(runs[0][0] + runs[0][1], Eo + Bo)
        log(f"wide tiles {dtype} solver {solver} {shape}: {max(e):.2e}")
        assert max(e) < (1e-12 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("shape", [(4, 30, 60), (6, 5, 62), (7, 20, 64), (3, 8, 124), (2, 25, 180)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_delta_form_norms_and_fields(shape, dtype):
    """The delta form's running sum and step norms over the same widths: the
    norm of dE' and the decisions as the oracle's, the fields at its counts."""
    w = _noise(shape, dtype, tol=1e-6 if dtype == "f32" else 1e-9)
    Ed, Bd, st, k = run_gpu(w, 2, form=mx.FORM_DELTA)
    _, _, so = run_oracle(w, 2, check_every=k)
    for a, b in zip(st, so):
        assert abs(a.sweeps[0] - b.sweeps[0]) <= k and a.sweeps[0] > 0
    assert st[0].rhs[0] == pytest.approx(so[0].rhs[0], rel=1e-12 if dtype == "f64" else 1e-6)
    Eo, Bo, _ = run_oracle(w, 2, replay=[s.sweeps for s in st])
    assert max(rel_err(Ed + Bd, Eo + Bo)) < (1e-12 if dtype == "f64" else 1e-5)
