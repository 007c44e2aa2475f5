"""The cut of the 3D sweep passes into workgroups (csrc/plan3d.h, host code):
every workgroup of a tolerance pass has a row of the partial sums that
mx_workspace_size counts, over wide, thin and ordinary boxes; rows whose byte
offsets need more than 32 bits are refused; the z chunks are those of trying
every count, found in a few microseconds however long the box is."""
import os
import shutil
import subprocess

import pytest

from paper_1907_13088_amd import mx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_13088_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "plan3d.h"
using namespace mx::plan3d;
int main() {
    int f64, nx, ny, nz, cus;
    while (std::scanf("%d %d %d %d %d", &f64, &nx, &ny, &nz, &cus) == 5) {
        long long most = 0;
        for (int k = 1; k <= kmax(f64); k++)
            for (const bool c : {false, true}) {   // the tiles launch_shape may take
                const bool lo = takes_low(f64, c, k, nx, ny, nz);
                for (const Shape s : {lo ? low(f64, c) : c ? cheb(f64) : large(f64), lo ? low(f64, c) : c ? cheb(f64) : small(f64)}) {
                    const Split p = split(s, k, nx, ny, nz, lo ? 2 * cus : cus);
                    most = std::max(most, (long long)p.gx * p.gy * p.nzc);
                }
            }
        std::printf("%lld %d\n", most, row_fits(nx, f64 ? 8 : 4));
    }
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("plan3d")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "driver"),
                    str(d / "driver.cpp")], check=True)
    return str(d / "driver")


def _rows(dtype, n):
    """Rows of two doubles behind the arrays and ahead of the solve's state in
    the workspace of a tolerance grid (arrays and areas in multiples of 256
    bytes; 21 arrays of Alg 1)."""
    up = lambda v: -(-v // 256) * 256
    c = mx.make_config(3, n, 0.3, (1.0, 1.0, 1.0), dtype, mx.MX_ALL, 20, 1e-6)
    arrays = 21 * up(n[0] * n[1] * n[2] * (8 if dtype == "f64" else 4))
    return (mx.workspace_size(c) - arrays - 256) // 16


def test_every_workgroup_has_a_row_of_partial_sums(driver):
    sizes = [(nx, ny, nz) for nx in (1, 57, 58, 59, 60, 61, 63, 64, 65, 940, 975, 1000, 3712, 5800, 37120, 100000)
             for ny in (1, 2, 3, 4, 5, 6, 7, 12, 13, 64) for nz in (1, 2, 3, 5, 64)]
    sizes += [(nx, 1, 1) for nx in range(900, 2200, 7)] + [(1000000, 3, 1), (256, 256, 256), (160, 144, 128)]
    cases = [(dtype, n, cus) for dtype in ("f32", "f64") for n in sizes for cus in (1, 256, 4096)]
    text = "".join(f"{int(d == 'f64')} {n[0]} {n[1]} {n[2]} {c}\n" for d, n, c in cases)
    out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(cases)
    for (dtype, n, cus), line in zip(cases, out):
        assert int(line.split()[0]) <= _rows(dtype, n), (dtype, n, cus, line)


def test_rows_of_4_gib_are_refused(driver):
    """The kernels keep a row's length in 32 bits of bytes: every width that
    mx_validate accepts is either swept with that length or refused."""
    cases = [(dtype, nx) for dtype in ("f32", "f64") for nx in (1, 4096, 2 ** 28, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 1, 2 ** 30)]
    text = "".join(f"{int(d == 'f64')} {nx} 1 1 256\n" for d, nx in cases)
    out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    for (dtype, nx), line in zip(cases, out):
        assert mx.validate(mx.make_config(3, (nx, 1, 1), 0.3, (1.0, 1.0, 1.0), dtype, mx.MX_ALL, 3)) == 0
        row = nx * (8 if dtype == "f64" else 4)
        assert (line.split()[1] == "1") == (row % 2 ** 32 == row), (dtype, nx)


SEARCH = r"""
#include <chrono>
#include <cstdio>
#include "plan3d.h"
using namespace mx::plan3d;
int main() {
    // every chunk count tried
    const int cus = 256;
    for (int nz : {1, 2, 3, 4, 5, 7, 16, 31, 64, 100, 128, 255, 512, 777, 1024, 3000})
        for (int nx : {1, 24, 58, 100, 160, 250, 512, 1000})
            for (int ny : {1, 12, 40, 144, 512})
                for (int f64 = 0; f64 < 2; f64++) {
                    for (int k = 1; k <= kmax(f64); k++)
                        for (const Shape s : {large(f64), small(f64), cheb(f64)}) {
                            const Split p = split(s, k, nx, ny, nz, cus);
                            const long long ncol = (long long)p.gx * p.gy;
                            double best = 1e300;
                            int bl = 0, bn = 0;
                            for (int n = 1; n <= std::max(1, nz / 2); n++) {
                                const int L = (nz + n - 1) / n, m = (nz + L - 1) / L;
                                const double c = (double)((ncol * m + cus - 1) / cus) * (L + 3 * k) * (s.nw * s.r + 8);
                                if (c < best * (1.0 - 1e-9)) best = c, bl = L, bn = m;
                            }
                            if (p.Lz != bl || p.nzc != bn) return std::printf("split %d %d %d\n", nx, ny, nz), 1;
                        }
                    for (int fill : {3, 4}) {
                        const long long ncol = (long long)((nx + 63) / 64) * ((ny + 7) / 8);
                        const Chunks c = front_chunks(ncol, nz, fill, 512);
                        double best = 1e300;
                        int bl = 0, bn = 0;
                        for (int n = 1; n <= std::max(1, nz / 2); n++) {
                            const int L = (nz + n - 1) / n, m = (nz + L - 1) / L;
                            const double t = (double)((ncol * m + 511) / 512) * (L + fill);
                            if (t < best * (1.0 - 1e-9)) best = t, bl = L, bn = m;
                        }
                        if (c.Lz != bl || c.nzc != bn) return std::printf("front %d %d %d\n", nx, ny, nz), 1;
                    }
                }
    // long boxes: microseconds per plan, the worst
    double worst = 0;
    for (int nz : {512, 4096, 65536, 1 << 20, 1 << 30})
        for (int nx : {1, 8, 64, 500}) {
            const auto t0 = std::chrono::steady_clock::now();
            volatile int sink = 0;
            for (int r = 0; r < 20; r++) {
                sink = sink + split(small(true), 1, nx, 8, nz, cus).Lz + split(large(false), 3, nx, 8, nz, cus).Lz;
                sink = sink + front_chunks((nx + 63) / 64, nz, 3, 1024).Lz;
            }
            const std::chrono::duration<double, std::micro> d = std::chrono::steady_clock::now() - t0;
            worst = std::max(worst, d.count() / 20);
        }
    std::printf("%.1f\n", worst);
}
"""


def test_the_search_for_z_chunks(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    (tmp_path / "search.cpp").write_text(SEARCH)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "search"),
                    str(tmp_path / "search.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "search")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    # three plans; trying every count takes 500 us at 65536 planes
    assert float(r.stdout) < 100, r.stdout
