"""The particle push at the edges of its paths: node fields formed once
(many particles), several particles per thread, deposition windows that cross
the periodic edge, windows too wide for the accumulation area; against the
FP64 oracle."""
import numpy as np
import pytest

from oracle import ref
from paper_1907_13088_amd import inputs as I
from paper_1907_13088_amd import mx

from gpu_helpers import log, to_np, torch_fields
from test_gpu_pic import _cell_order, _gpu_state, _rel, _setup

pytestmark = pytest.mark.gpu


def _shifted(sp, d, shape, sx, sy):
    """Cell order of the box shifted by (sx, sy): workgroups straddle its edges."""
    ny, nx = shape
    cx = (np.floor(sp.x / d[0]).astype(np.int64) + sx) % nx
    cy = (np.floor(sp.y / d[1]).astype(np.int64) + sy) % ny
    o = np.argsort(cy * nx + cx, kind="stable")
    return I.Species(q=sp.q, m=sp.m, w=sp.w, x=sp.x[o].copy(), y=sp.y[o].copy(), u=[a[o].copy() for a in sp.u])


@pytest.mark.parametrize("shape,dtype,npart,order", [
    ((29, 37), "f64", 262143, "cell"), ((29, 37), "f64", 262145, "cell"),     # node fields from 2^18 particles
    ((29, 37), "f64", 1100003, "cell"), ((29, 37), "f32", 300000, "cell"),    # two per thread
    ((29, 37), "f64", 60000, "shifted"), ((12, 9), "f64", 280000, "shifted"),
    ((3, 2), "f64", 5000, "random"), ((300, 210), "f64", 40000, "cell"), ((300, 210), "f64", 140000, "shifted"),
    ((260, 250), "f64", 270000, "random"), ((29, 37), "f64", 1, "cell"), ((29, 37), "f64", 257, "shifted")])
def test_push_and_deposition_paths(shape, dtype, npart, order):
    import torch
    d = (0.9, 1.2)
    cfg_o, cfg_g, E, B, species = _setup(shape, d, dtype, seed=5, nspec=1, npart=max(npart, 3))
    sp = species[0]
    if npart < 3:
        sp = I.Species(q=sp.q, m=sp.m, w=sp.w, x=sp.x[:npart], y=sp.y[:npart], u=[a[:npart] for a in sp.u])
    if order == "cell":
        sp = _cell_order(sp, d, shape[1])
    elif order == "shifted":
        sp = _shifted(sp, d, shape, shape[1] // 2, shape[0] // 2)
    g = mx.Grid(cfg_g)
    g.bind(torch_fields(E, dtype), torch_fields(B, dtype))
    Jt = [torch.full(shape, 7.0, dtype=g.torch_dtype, device="cuda") for _ in range(3)]
    pos, u = _gpu_state(sp, dtype)
    g.pic_push(sp.q, sp.m, sp.w, pos, u, Jt)
    Jo = [np.zeros(shape) for _ in range(3)]
    xo, yo, uo = sp.x.copy(), sp.y.copy(), [a.copy() for a in sp.u]
    ref.pic_push_deposit(cfg_o, E, B, sp.q, sp.m, sp.w, xo, yo, *uo, Jo)
    torch.cuda.synchronize()
    g.close()
    e_j = _rel(to_np(Jt), Jo)
    log(f"{shape} {dtype} {npart} {order}: current {e_j:.2e}")
    if dtype == "f64":
        # the same operations in the same order: positions and momenta bitwise
        for a, b in zip(to_np(pos) + to_np(u), [xo, yo] + uo):
            assert np.array_equal(a, b)
        assert e_j <= 1e-12
    else:
        # a position near 40 has an ulp of 4e-6 and a move is about 0.3 cells:
        # about 1e-5 per contribution
        assert e_j <= 1e-4 and _rel(to_np(u), uo) <= 1e-6
