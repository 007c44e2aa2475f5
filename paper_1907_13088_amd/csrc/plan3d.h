#pragma once
// How a 3D sweep pass (k3s.hip) is cut into workgroups, and how many rows of
// partial sums that takes.  Host code without HIP, so that the workspace, the
// launch and a CPU test go by the same rules.
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace mx {
namespace plan3d {

// deepest pass
constexpr int kmax(bool f64) { return f64 ? 2 : 3; }

// A row of the grid is one buffer of 32-bit byte offsets, the last of which
// (0xffffffff) stands for "no cell"
constexpr bool row_fits(int64_t nx, size_t elem) { return nx * (int64_t)elem <= 0xffffffffLL; }

// Tiles: R rows per wave, NW waves: the larger and the smaller one of Alg 1 and
// the delta form, that of the Chebyshev form, and the lowest ones for boxes of
// few rows or planes
struct Shape {
    int r, nw;
};
constexpr Shape large(bool f64) { return {2, f64 ? 8 : 12}; }
constexpr Shape small(bool f64) { return {2, f64 ? 4 : 8}; }
constexpr Shape cheb(bool f64) { return {1, f64 ? 12 : 16}; }
constexpr Shape low(bool f64, bool cheb) { return f64 && cheb ? Shape{1, 8} : Shape{2, 4}; }

// A launch's z chunks and its time in the model that sizes it: a workgroup
// marches Lz + 3K plane steps (its chunk and the pipeline's fill and drain),
// the workgroups run in rounds of one per CU, and a step costs its rows plus
// about 8 (the barrier and the latencies of a step on a CU that is not full;
// fitted on 64^3 to 512^3).  Chunks of two planes pay on small grids, where
// they are what fills the CUs.
struct Split {
    int gx, gy, Lz, nzc;
    double cost;
    bool wide;            // tiles two columns wider, at some work per step
};

// output columns and rows of a tile in a pass of k sweeps
constexpr int out_x(int k, bool wide) { return 64 - 2 * (wide ? k - 1 : k); }
constexpr int out_y(Shape s, int k) { return s.nw * s.r - 2 * (k - 1); }

// a wide tile's step against a narrow one's (measured 1.03 to 1.07)
constexpr double WIDE_COST = 1.08;
inline Split split_of(Shape s, int k, bool wide, int nx, int ny, int nz, int cus)
{
    const int ox = out_x(k, wide), oy = out_y(s, k);
    Split best{(nx + ox - 1) / ox, (ny + oy - 1) / oy, nz, 1, 1e300, wide};
    const int64_t ncol = (int64_t)best.gx * best.gy;
    // (more chunks only add fills and drains once the CUs are shared evenly, so
    // the search ends after some hundreds of steps however long the box is)
    for (int n = 1; n <= std::max(1, nz / 2); n++) {
        const int Lz = (nz + n - 1) / n, nzc = (nz + Lz - 1) / Lz;
        if ((double)ncol * (nz + 3.0 * k * nzc) / cus * (s.nw * s.r + 8) >= best.cost) break;   // below any cost from here on
        const double cost = (double)((ncol * nzc + cus - 1) / cus) * (Lz + 3 * k) * (s.nw * s.r + 8);
        if (cost < best.cost * (1.0 - 1e-9)) best.cost = cost, best.Lz = Lz, best.nzc = nzc;
    }
    return best;
}

// Wide tiles where they save columns of tiles
inline Split split(Shape s, int k, int nx, int ny, int nz, int cus)
{
    Split n = split_of(s, k, false, nx, ny, nz, cus);
    if ((nx + out_x(k, true) - 1) / out_x(k, true) == n.gx) return n;
    Split w = split_of(s, k, true, nx, ny, nz, cus);
    w.cost *= WIDE_COST;
    return w.cost < n.cost ? w : n;
}

// z chunks of the 3D front (k3f.hip): every workgroup marches its chunk and
// `fill` plane steps that fill the z filter and the B planes below it, in rounds
// of the `slots` resident workgroups; the count with the fewest plane steps.
struct Chunks {
    int Lz, nzc;
};
inline Chunks front_chunks(int64_t ncol, int nz, int fill, int slots)
{
    Chunks best{nz, 1};
    double least = 1e300;
    for (int n = 1; n <= std::max(1, nz / 2); n++) {
        const int L = (nz + n - 1) / n, m = (nz + L - 1) / L;
        if ((double)ncol * (nz + (double)fill * m) / slots >= least) break;   // as above
        const double steps = (double)((ncol * m + slots - 1) / slots) * (L + fill);
        if (steps < least * (1.0 - 1e-9)) least = steps, best = Chunks{L, m};
    }
    return best;
}

// Boxes of one or two planes run passes of single sweeps: the pipeline's fill
// and drain, three plane steps per sweep of the pass, are most of a march
// (1024 x 1024 x 1, six Chebyshev sweeps, FP32 359 us per step in passes of three, 250 so).
constexpr bool flat(int64_t nz) { return nz <= 2; }
// The lowest tiles, for the passes of flat boxes and where the rows of a box fill
// one of them, in wide boxes little more (a taller tile is mostly padding then;
// us per step, FP32, lowest against taller tiles: 1024 x 1 x 1024 delta form 1093 against 2387, 65536 x 8
// x 8 Alg 1 397 against 551, 200000 x 4 x 1 Chebyshev 335 against 691; 8 x 8 x 65536
// Chebyshev 2320 against 2016).
inline bool takes_low(bool f64, bool cheb, int k, int64_t nx, int64_t ny, int64_t nz)
{
    return (flat(nz) && k == 1) || ny <= (nx > 64 && !f64 ? 8 : out_y(low(f64, cheb), k));
}

// Rows of partial sums (one per workgroup) of any pass on this grid, whatever
// the number of CUs: the tiles of the narrowest and lowest output, times the
// most chunks.
inline int64_t partial_rows(bool f64, int64_t nx, int64_t ny, int64_t nz)
{
    int64_t rows = 0;
    for (int k = 1; k <= kmax(f64); k++) {
        auto count = [&](Shape s) {
            const int ox = out_x(k, false), oy = out_y(s, k);
            rows = std::max(rows, ((nx + ox - 1) / ox) * ((ny + oy - 1) / oy) * std::max<int64_t>(1, nz / 2));
        };
        count(large(f64)), count(small(f64)), count(cheb(f64));
        for (const bool c : {false, true})
            if (takes_low(f64, c, k, nx, ny, nz)) count(low(f64, c));
    }
    return rows;
}

}  // namespace plan3d
}  // namespace mx
