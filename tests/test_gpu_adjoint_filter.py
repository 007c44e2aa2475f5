"""The current gradient of the transposed step: its filter in one launch."""
import numpy as np
import pytest

from oracle import ref

from gpu_helpers import log, to_np, torch_fields
from test_gpu_adjoint import _grid

pytestmark = pytest.mark.gpu


# a wave writes (64 - 2p) x 24 cells; shapes at, under and over that tile
# and smaller than the rim
@pytest.mark.parametrize("p", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("shape", [(3, 5), (24, 58), (25, 57), (97, 130)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_current_gradient_filter(p, shape, dtype):
    """Three transposed steps that add to a current gradient in hand, the last
    step (the first one backwards) with a zero envelope: within 1e-12 (FP64)
    or 2e-6 (FP32: some tens of roundings of 6e-8) of the oracle; a block that
    is not stepped leaves its gradient as it was."""
    rng = np.random.default_rng(70 + p)
    envs, m = [0.7, -0.4, 0.0], 2
    rnd = lambda: [rng.normal(size=shape).astype(np.float32).astype(np.float64) for _ in range(3)]
    Eb, Bb, J = rnd(), rnd(), rnd()
    cfg = ref.Config(ndim=2, shape=shape, dt=0.3, sweeps=m, filter_passes=p)
    Eo, Bo, Jo = [[a.copy() for a in f] for f in (Eb, Bb, J)]
    for n in (2, 1, 0):
        ref.adjoint_step(cfg, Eo, Bo, Jo, envs[n], (m, m))
    for blocks in (3, 1):
        g = _grid(2, shape, 0.3, dtype, m, p, blocks=blocks)
        Et, Bt, Jt = [torch_fields(f, dtype) for f in (Eb, Bb, J)]
        g.adjoint(3, envs, [(m, m)] * 3, Et, Bt, Jt)
        got = to_np(Jt)
        want = Jo if blocks == 3 else Jo[:2] + [J[2]]
        scale = max(np.abs(x).max() for x in want)
        err = max(np.abs(a - b).max() for a, b in zip(got, want)) / scale
        log(f"current gradient {dtype} p={p} {shape} blocks {blocks}: {err:.2e}")
        assert err < (1e-12 if dtype == "f64" else 2e-6)
