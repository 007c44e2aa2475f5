"""Register-tile passes (the library's choice for fixed counts on grids of up
to a few million cells) against the row-streaming and LDS-tile kernels: every
schedule forms each value by the same operations, so fields are bitwise
equal, over tile edges and remainders, every tile geometry, filter depths,
odd and even step counts (the last step hands B back) and counts that differ
per block and step."""
import numpy as np
import pytest

from paper_1907_13088_amd import mx

pytestmark = pytest.mark.gpu


def _rand(shape, dtype, seed, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    td = torch.float64 if dtype == "f64" else torch.float32
    return [torch.randn(shape, generator=g, dtype=torch.float64, device="cuda").to(td) for _ in range(n)]


def _run(n, dtype, variant, m, p, steps, blocks=mx.MX_ALL, replay=None, current=True, lumped=False, d=(1.0, 1.0)):
    import torch
    dt = 0.45 / (1 / d[0] ** 2 + 1 / d[1] ** 2) ** 0.5
    g = mx.Grid(mx.make_config(2, n, dt, d, dtype, blocks, m, 0.0, p, variant=variant, lumped=lumped))
    f = _rand((n[1], n[0]), dtype, 7, 9)
    g.bind(f[:3], f[3:6])
    if current:
        g.set_current(f[6:])
    env = [0.7 - 0.3 * s for s in range(sum(steps))]
    at = 0
    st = []
    for k in steps:
        st += g.step(k, env=env[at:at + k], replay=None if replay is None else replay[at:at + k], stats=True)
        at += k
    torch.cuda.synchronize()
    g.close()
    return f[:6], [s.sweeps for s in st]


def _same(a, b, what):
    import torch
    for q, (x, y) in enumerate(zip(a[0], b[0])):
        assert torch.equal(x, y), (what, q, (x - y).abs().max().item())
    assert a[1] == b[1], what


SIZES = [(1, 1), (2, 3), (5, 70), (31, 17), (64, 32), (44, 12), (45, 13), (129, 65), (300, 257), (700, 300)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", SIZES)
def test_sizes_and_remainders(n, dtype):
    for m, p, steps in ((20, 3, (3,)), (1, 0, (1, 1)), (7, 4, (2,))):
        _same(_run(n, dtype, 0, m, p, steps), _run(n, dtype, 2, m, p, steps), (n, dtype, m, p))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("blocks", [mx.MX_TE, mx.MX_TM, mx.MX_ALL])
@pytest.mark.parametrize("n", [(96, 80), (512, 500), (1030, 1000), (1500, 1101)])
def test_every_geometry_and_block_set(n, blocks, dtype):
    # the plan takes 64 x 32, 64 x 64 and 128 x 64 regions over these sizes
    for m, p, d in ((20, 1, (1.0, 1.0)), (9, 2, (0.8, 1.3))):
        _same(_run(n, dtype, 0, m, p, (2,), blocks, d=d), _run(n, dtype, 3, m, p, (2,), blocks, d=d), (n, blocks, m))


@pytest.mark.parametrize("m", [0, 2, 3, 13, 14, 15, 29, 61])
def test_counts(m):
    for current in (True, False):
        _same(_run((210, 90), "f32", 0, m, 2, (3, 1), current=current),
              _run((210, 90), "f32", 1, m, 2, (3, 1), current=current), m)
    _same(_run((210, 90), "f64", 0, m, 2, (2,), lumped=True), _run((210, 90), "f64", 3, m, 2, (2,), lumped=True), m)


def test_counts_per_block_and_step():
    counts = [(0, 5), (17, 0), (1, 33), (23, 2), (0, 0), (10, 10), (20, 20)]
    for dtype in ("f32", "f64"):
        _same(_run((333, 120), dtype, 0, 20, 3, (4, 3), replay=counts),
              _run((333, 120), dtype, 3, 20, 3, (4, 3), replay=counts), dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_transposed_steps(dtype):
    import torch
    n, counts = (333, 120), [(20, 20), (3, 0), (0, 9), (20, 20)]
    out = []
    for variant in (0, 3):
        g = mx.Grid(mx.make_config(2, n, 0.3, (1.0, 1.0), dtype, mx.MX_ALL, 20, 0.0, 2, variant=variant))
        f = _rand((n[1], n[0]), dtype, 11, 9)
        g.adjoint(4, [0.3, -0.2, 0.0, 0.9], counts, f[:3], f[3:6], f[6:])
        torch.cuda.synchronize()
        g.close()
        out.append((f, None))
    _same(out[0], out[1], dtype)


def test_a_caller_stream_and_graph_replays():
    """Plain launches only: a captured step replays on the caller's stream
    like the eager one."""
    import torch
    n = (257, 130)
    s = torch.cuda.Stream()
    cfg = mx.make_config(2, n, 0.4, (1.0, 1.0), "f32", mx.MX_ALL, 20, 0.0, 2)
    f = _rand((n[1], n[0]), "f32", 3, 9)
    e = [t.clone() for t in f]
    torch.cuda.synchronize()
    g, g2 = mx.Grid(cfg, stream=s), mx.Grid(cfg)
    g.bind(f[:3], f[3:6])
    g.set_current(f[6:])
    g2.bind(e[:3], e[3:6])
    g2.set_current(e[6:])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.step(3, env=[0.1, 0.2, 0.3])
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        g2.step(3, env=[0.1, 0.2, 0.3])
        torch.cuda.synchronize()
        for x, y in zip(f[:6], e[:6]):
            assert torch.equal(x, y)
    g.close()
    g2.close()
