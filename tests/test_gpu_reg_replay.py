"""Chebyshev steps on register tiles whose counts differ from step to step of
one call: a step of more than two passes keeps an iterate where the filtered
current stood, and the next front has to read the current all the same."""
import pytest

from paper_1907_13088_amd import mx

from test_gpu_reg import _rand, _same

pytestmark = pytest.mark.gpu


# counts on both sides of the cut into two and three passes (on 512^2 both
# blocks: 17 sweeps), of one block and of both, falling and rising
@pytest.mark.parametrize("n,counts,blocks", [
    ((512, 512), [(20, 20), (7, 7), (20, 9), (5, 20), (7, 7), (40, 40), (3, 3)], mx.MX_ALL),
    ((512, 512), [(12, 0), (4, 0), (25, 0), (10, 0)], mx.MX_TE),
    ((333, 120), [(0, 30), (0, 5), (0, 61), (0, 2)], mx.MX_TM),
    ((1500, 1100), [(16, 16), (6, 6), (2, 30), (6, 6)], mx.MX_ALL)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_counts_that_cross_the_pass_limit(n, counts, blocks, dtype):
    import torch
    env = [0.7 - 0.2 * s for s in range(len(counts))]
    out = []
    for variant in (0, 3):
        g = mx.Grid(mx.make_config(2, n, 0.35, (1.0, 1.0), dtype, blocks, 7, 0.0, 2, variant=variant, solver=1))
        f = _rand((n[1], n[0]), dtype, 21, 9)
        g.bind(f[:3], f[3:6])
        g.set_current(f[6:])
        st = g.step(len(counts), env=env, replay=counts, stats=True)
        torch.cuda.synchronize()
        g.close()
        out.append((f, [s.sweeps for s in st]))
    _same(out[0], out[1], (n, counts, dtype))
