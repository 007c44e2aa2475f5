"""Which 2D solves take register tiles (csrc/plan2r.h, host code): on grids
measured on both kernels, the faster one."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_13088_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "plan2r.h"
using namespace mx;
int main() {
    char what;
    int f64, blocks, cheb, nx, ny, m, u, v;
    while (std::scanf(" %c %d %d %d %d %d %d %d %d", &what, &f64, &blocks, &cheb, &nx, &ny, &m, &u, &v) == 9) {
        int yes = 0;
        if (what == 'f')   // fixed counts: u steps, v filtered current
            yes = reg_pays(reg_plan(f64, blocks, cheb, true, nx, ny, m), f64, blocks, cheb, true, nx, ny, m, u, v);
        else if (what == 'a')   // transposed solve
            yes = reg_pays(reg_plan(f64, blocks, cheb, false, nx, ny, m), f64, blocks, cheb, false, nx, ny, m, 1, false);
        else if (what == 't') {   // tolerance solve: tested passes of m sweeps, u delta form, v norms per block
            const RegPlan p = reg_tol_plan(f64, blocks, cheb, nx, ny, m, v);
            yes = reg_tol_pays(p, f64, blocks, cheb, u, nx, ny, m);
        } else {   // batch of u grids
            mx_config c{};
            c.dtype = f64 ? MX_F64 : MX_F32;
            c.sweeps = m;
            c.n[0] = nx;
            c.n[1] = ny;
            std::vector<mx_config> all(u, c);
            yes = reg_batch_plan(all.data(), u).geo >= 0;
        }
        std::printf("%d\n", yes);
    }
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("plan2r")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "driver"),
                    str(d / "driver.cpp")], check=True)

    def run(lines):
        text = "".join(" ".join(str(int(x) if isinstance(x, bool) else x) for x in l) + "\n" for l in lines)
        out = subprocess.run([str(d / "driver")], input=text, capture_output=True, text=True, check=True).stdout.split()
        assert len(out) == len(lines)
        return [o == "1" for o in out]
    return run


def _fixed(f64, nx, ny, m=20, steps=8, filt=True, blocks=3, cheb=False):
    return ("f", f64, blocks, cheb, nx, ny, m, steps, filt)


def _tol(f64, nx, ny, k=8, delta=False, blocks=3, cheb=False):
    rows = max(-(-nx // 64) * -(-ny // 4), (-(-nx // 224) + 1) * ny)
    return ("t", f64, blocks, cheb, nx, ny, k, delta, rows // 3)


def _batch(f64, ng, nx, ny, m=20):
    return ("b", f64, 3, 0, nx, ny, m, ng, 0)


def test_ordinary_grids(tiles):
    yes = [_fixed(f, *n) for f in (0, 1) for n in ((64, 48), (700, 300), (1024, 1024), (1500, 1100), (2048, 1450))]
    yes += [_tol(f, *n) for f in (0, 1) for n in ((64, 48), (700, 300), (1024, 1024), (1500, 1100))]
    yes += [_batch(f, 8, 1464, 256) for f in (0, 1)] + [_batch(f, 64, 64, 244) for f in (0, 1)]
    no = [_fixed(f, 4096, 4096) for f in (0, 1)] + [_tol(f, 2560, 2048) for f in (0, 1)]
    assert tiles(yes) == [True] * len(yes)
    assert tiles(no) == [False] * len(no)


def test_thin_grids(tiles):
    """Grids whose short side holds little of a tile: streamed where the
    padding costs more than the latency saved."""
    no = [_fixed(f, *n) for f in (0, 1) for n in ((3000000, 1), (1500000, 2), (750000, 4), (1000000, 1), (500000, 2))]
    no += [_fixed(0, 46875, 64), _fixed(0, 1000000, 1, m=8, cheb=True), _fixed(0, 250000, 4, m=8, cheb=True)]
    no += [("a", f, 3, 0, *n, 20, 0, 0) for f in (0, 1) for n in ((3000000, 1), (750000, 4), (1000000, 1))]
    no += [_tol(0, *n) for n in ((1, 3000000), (2, 1500000), (4, 750000), (375000, 8), (46875, 64), (187500, 16),
                                 (125000, 8))]
    no += [_tol(1, *n) for n in ((1, 3000000), (46875, 64), (187500, 16))]
    no += [_tol(1, *n, k=4, cheb=True) for n in ((1, 1000000), (2, 500000), (4, 250000))]
    no += [_batch(f, ng, n // ng, s) for f in (0, 1) for ng in (8, 64)
           for n, s in ((3000000, 1), (1500000, 2), (750000, 4), (1000000, 1), (500000, 2), (250000, 4), (200000, 1),
                        (100000, 2))]
    no += [_batch(0, 8, 46875, 8), _batch(0, 8, 15625, 8)]
    yes = [_fixed(f, *n) for f in (0, 1) for n in ((1, 3000000), (16, 187500), (64, 46875), (187500, 16), (1, 60000),
                                                   (30000, 2), (15000, 4), (7500, 8))]
    yes += [_tol(f, *n) for f in (0, 1) for n in ((64, 40000), (62500, 16), (64, 15625), (1, 60000), (3750, 16))]
    yes += [_batch(f, 8, *n) for f in (0, 1) for n in ((1, 125000), (16, 7812), (7812, 16), (3125, 8), (1562, 16))]
    got = tiles(no)
    assert not any(got), [l for l, g in zip(no, got) if g]
    got = tiles(yes)
    assert all(got), [l for l, g in zip(yes, got) if not g]


def test_few_sweeps_and_short_calls(tiles):
    """A step of few sweeps, and one that pays the current's filter alone,
    leaves the tiles little to win."""
    no = [_fixed(0, 2048, 1450, m=3), _fixed(0, 2048, 1600, m=6), _fixed(1, 1500, 1400, m=3), _fixed(1, 2048, 2048, m=3),
          _fixed(1, 1500, 1400, m=6), _fixed(1, 2048, 2048, m=3, blocks=1), _fixed(1, 2048, 1600, m=6, blocks=1),
          _fixed(1, 1500, 1100, m=3, steps=1), _fixed(1, 1500, 1400, m=6, steps=1), _fixed(0, 1500, 1400, m=3, steps=1),
          _fixed(0, 1500, 1400, m=3, steps=1, blocks=1), _fixed(1, 2048, 1450, m=0, filt=False),
          _fixed(1, 1500, 1100, m=3, cheb=True), _fixed(1, 1024, 1000, m=3, steps=1, cheb=True),
          _fixed(1, 1500, 1100, m=7, steps=1, cheb=True), _fixed(0, 1500, 1400, m=3, cheb=True),
          _fixed(0, 1500, 1400, m=3, steps=1, cheb=True), _batch(0, 5, 900, 600, m=2), _batch(1, 8, 700, 400, m=3),
          _batch(1, 8, 1000, 900, m=3)]
    yes = [_fixed(0, 1500, 1100, m=8, steps=1), _fixed(0, 2048, 1600, m=20), _fixed(1, 2048, 2048, m=20),
           _fixed(1, 2048, 1600, m=8), _fixed(0, 2048, 2048, m=20, blocks=1), _fixed(1, 1024, 1000, m=7, cheb=True),
           _fixed(0, 1500, 1100, m=7, cheb=True), _fixed(0, 500, 400, m=3, steps=1), _fixed(1, 500, 400, m=3, steps=1),
           _batch(0, 8, 500, 256, m=2), _batch(1, 8, 1000, 900, m=5), _batch(1, 8, 500, 256, m=3)]
    yes += [("a", f, b, 0, 2048, 2048 if f else 1600, m, 0, 0) for f in (0, 1) for b in (1, 3) for m in (1, 3, 20)]
    got = tiles(no)
    assert not any(got), [l for l, g in zip(no, got) if g]
    got = tiles(yes)
    assert all(got), [l for l, g in zip(yes, got) if not g]


def test_delta_form_tolerance_solves(tiles):
    """The delta form's passes move the running sum too: streamed from smaller
    grids on, in FP64 above all."""
    no = [_tol(1, *n, delta=True) for n in ((1500, 1400), (1800, 1300), (2048, 1450), (2048, 1600))]
    no += [_tol(1, 2048, 1450, delta=True, blocks=b) for b in (1, 2)]
    no += [_tol(0, 2048, 1600, delta=True), _tol(1, 2048, 1450)]
    yes = [_tol(1, *n, delta=True) for n in ((700, 300), (1024, 1024), (1500, 1100))]
    yes += [_tol(1, 1500, 1400, delta=True, blocks=b) for b in (1, 2)]
    yes += [_tol(0, 2048, 1450, delta=True), _tol(0, 2048, 1600), _tol(1, 1800, 1300), _tol(1, 2048, 1600, blocks=1)]
    got = tiles(no)
    assert not any(got), [l for l, g in zip(no, got) if g]
    got = tiles(yes)
    assert all(got), [l for l, g in zip(yes, got) if not g]
