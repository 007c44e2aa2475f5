#pragma once
// Which 2D solves run on register tiles (k2r_impl.h), on which tiles and in how
// many passes.  Host code without HIP, so that a CPU test goes by the same
// rules.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/mx.h"

namespace mx {

enum : int { RK_FRONT = 0, RK_MID = 1, RK_LAST = 2 };   // kinds of pass

// How one solve of m sweeps of a block set is cut: the tile geometry and the
// number of passes (front + others when `front`, else passes without one)
struct RegPlan {
    int geo, passes;
    double us;            // modelled time
};
// The same for the grids of a batch, both blocks, fixed counts.  kf: sweeps of
// the front's pass; ks: of the deepest other
struct RegBatchPlan {
    int geo, passes, kf, ks;
};

namespace reg2d {

// Tile geometries: columns and rows of the region.  Two neighbouring columns
// per lane (FP32) halve the lane shifts and widen the region; in FP64 they
// leave a CU one workgroup, and nothing hides its loads (1500 x 1100, 8
// sweeps, TE 72 against 41 us).
struct Geo {
    int rx, ry;
};
inline constexpr Geo GEO[4] = {{64, 32}, {64, 32}, {64, 64}, {128, 64}};

// Time of a pass (us) with c workgroups per CU: t0 + c load[kind] + k (c s + s0),
// fitted to single passes over grids from 128^2 to 2048^2, every kind, depths 0, 2,
// 4, 6, 8, 10 and 14, every geometry, each block alone and both in one launch:
// per form, type, blocks and geometry one non-negative least-squares fit of the
// six numbers to the measured times, each divided by its time (rms 5 to 20 %;
// the choice it makes is within 3 % of the best measured one on average, 35 %
// at worst).  By form (standard and delta, Chebyshev), type and blocks,
// geometry.
struct Fit {
    double t0, load[3], s, s0;
};
inline constexpr Fit FIT[2][6][4] = {
    {
     {{2.65, {1.72, 1.37, 1.75}, 0.131, 0.069},
      {3.18, {1.46, 0.98, 1.58}, 0.066, 0.145},
      {1.39, {3.50, 2.72, 3.93}, 0.166, 0.270},
      {1.23, {9.68, 6.70, 9.25}, 0.084, 0.695}},   // FP32 TE
     {{3.07, {1.45, 0.77, 1.00}, 0.146, 0.028},
      {3.45, {1.18, 0.51, 0.75}, 0.090, 0.056},
      {2.68, {2.54, 1.30, 1.90}, 0.222, 0.092},
      {2.05, {8.25, 3.23, 4.53}, 0.177, 0.414}},   // FP32 TM
     {{2.28, {1.79, 1.40, 1.89}, 0.107, 0.122},
      {2.69, {1.65, 1.12, 1.71}, 0.041, 0.198},
      {1.39, {3.68, 2.73, 3.97}, 0.148, 0.273},
      {1.34, {9.42, 6.70, 8.93}, 0.104, 0.655}},   // FP32 both
     {{2.21, {3.56, 2.77, 3.42}, 0.127, 0.173},
      {2.44, {3.28, 2.51, 3.35}, 0.027, 0.302},
      {0.02, {7.36, 5.97, 7.52}, 0.144, 0.467}},   // FP64 TE
     {{3.36, {2.52, 1.23, 1.51}, 0.189, 0.081},
      {3.52, {2.66, 1.04, 1.34}, 0.105, 0.176},
      {2.05, {6.10, 2.60, 3.42}, 0.259, 0.221}},   // FP64 TM
     {{2.03, {3.61, 2.73, 3.37}, 0.089, 0.230},
      {2.20, {3.63, 2.63, 3.38}, 0.003, 0.312},
      {0.00, {7.81, 5.94, 7.31}, 0.130, 0.457}},   // FP64 both
    },
    {
     {{2.16, {2.45, 2.18, 2.38}, 0.152, 0.197},
      {2.75, {2.06, 1.78, 2.20}, 0.091, 0.264},
      {0.38, {4.81, 4.56, 5.47}, 0.251, 0.442},
      {0.00, {13.02, 12.34, 13.38}, 0.949, 0.189}},   // FP32 TE
     {{2.96, {1.74, 1.14, 1.22}, 0.167, 0.085},
      {3.32, {1.47, 0.80, 0.95}, 0.098, 0.152},
      {2.28, {3.17, 2.23, 2.40}, 0.251, 0.199},
      {0.00, {11.32, 7.38, 7.96}, 0.592, 0.191}},   // FP32 TM
     {{1.98, {2.53, 2.16, 2.49}, 0.122, 0.211},
      {2.48, {2.25, 1.86, 2.27}, 0.071, 0.268},
      {0.19, {5.28, 4.65, 5.51}, 0.206, 0.475},
      {0.00, {13.34, 12.44, 13.20}, 0.960, 0.130}},   // FP32 both
     {{1.11, {5.32, 4.98, 5.03}, 0.063, 0.371},
      {0.97, {5.35, 5.00, 5.58}, 0.000, 0.468},
      {0.00, {9.01, 8.50, 9.20}, 0.868, 0.000}},   // FP64 TE
     {{2.90, {3.24, 2.12, 2.07}, 0.167, 0.217},
      {2.99, {3.26, 2.08, 2.36}, 0.109, 0.207},
      {0.00, {8.02, 6.00, 6.17}, 0.534, 0.069}},   // FP64 TM
     {{1.00, {5.05, 4.48, 4.60}, 0.054, 0.411},
      {0.71, {5.12, 4.57, 5.28}, 0.016, 0.474},
      {0.00, {9.42, 8.75, 9.27}, 0.806, 0.000}},   // FP64 both
    }};

// workgroups per CU of a launch of n: whole ones while they are few
inline double per_cu(double n) { return n <= 1024 ? std::ceil(n / 256) : n / 256 + 0.5; }

// workgroups per block of a pass
inline int64_t tiles(const Geo &g, int kind, int k, int64_t nx, int64_t ny)
{
    const int W = g.rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = g.ry - 2 * k;
    return ((nx + W - 1) / W) * ((ny + H - 1) / H);
}

inline double pass_us(const Fit &f, const Geo &g, int blocks, int kind, int k, int64_t nx, int64_t ny)
{
    const int W = g.rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = g.ry - 2 * k;
    if (W < 12 || H < 4) return 1e30;
    const double c = per_cu((double)tiles(g, kind, k, nx, ny) * (blocks == 3 ? 2 : 1));
    return f.t0 + c * f.load[kind] + k * (c * f.s + f.s0);
}

// Row streams against the time `us` modelled for the tiles.  At the limit, a
// square of `most` cells, both take `meet`; of that a part `a` is latency,
// which a grid of fewer cells pays too, and the rest goes with the cells of the
// streams' strips of `w` columns (narrow grids leave much of a strip empty)
// and with the rows that fill a chunk, felt as `fill` more rows (thin grids).
inline double strip_cells(int64_t nx, int64_t ny, int w, int fill) { return (double)((nx + w - 1) / w * w) * (double)(ny + fill); }
inline bool tiles_win(double us, double meet, double a, double strips, int64_t most)
{
    return us <= meet * (a + (1.0 - a) * strips / (double)most);
}
// Asked where a side is shorter than this; else the limit decides.  (A few
// tiles: with six or more along each side the last one's padding is small.)
constexpr int64_t SHORT = 256;
inline int64_t side_of(int64_t cells) { return (int64_t)std::sqrt((double)cells); }

}  // namespace reg2d

inline RegPlan reg_plan(bool f64, int blocks, bool cheb, bool front, int64_t nx, int64_t ny, int m)
{
    using namespace reg2d;
    RegPlan best{-1, 0, 1e29};
    const Fit *fit = FIT[cheb][(f64 ? 3 : 0) + blocks - 1];
    for (int g = 0; g < (f64 ? 3 : 4); g++) {
        const int kmax = std::min((GEO[g].ry - 4) / 2, 16);   // 16: the factor table of a pass
        const int n0 = std::max(front ? 2 : 1, (m + kmax - 1) / kmax);
        for (int n = n0; n <= n0 + 6; n++) {
            double t = 0.0;
            for (int i = 0, rem = m; i < n; i++) {
                const int k = rem / (n - i);
                const int kind = front && i == 0 ? RK_FRONT : (front && i == n - 1 ? RK_LAST : RK_MID);
                t += pass_us(fit[g], GEO[g], blocks, kind, k, nx, ny);
                rem -= k;
            }
            if (t < best.us) best = RegPlan{g, n, t};
        }
    }
    return best;
}

// geometry of a tolerance solve whose tested passes have k sweeps, in
// launches of nearly equal depth, with at most `stride` workgroups per block
// (geo < 0: none); passes: launches of a tested pass
inline RegPlan reg_tol_plan(bool f64, int blocks, bool cheb, int64_t nx, int64_t ny, int k, int64_t stride)
{
    using namespace reg2d;
    RegPlan best{-1, 0, 1e29};
    const Fit *fit = FIT[cheb][(f64 ? 3 : 0) + blocks - 1];
    for (int g = 0; g < (f64 ? 3 : 4); g++) {
        const int kmax = std::min((GEO[g].ry - 4) / 2, 16);   // 16: the factor table of a pass
        const int n0 = (k + kmax - 1) / kmax;
        for (int n = n0; n <= n0 + 1; n++) {
            // two tested passes, the first with the front
            double t = 0.0;
            bool fits = true;
            for (int i = 0; i < 2 * n; i++) {
                const int kind = i == 0 ? RK_FRONT : RK_MID, kk = (k + n - 1) / n;
                t += pass_us(fit[g], GEO[g], blocks, kind, kk, nx, ny);
                fits = fits && tiles(GEO[g], kind, kk, nx, ny) <= stride;
            }
            if (fits && t < best.us) best = RegPlan{g, n, t};
        }
    }
    return best;
}

// Register tiles against row streams, us per step.
// Fixed counts (20 sweeps, current, filter), FP32: both blocks 1024^2 64
// against 130, 2048 x 1600 163 against 178, 2048^2 217 against 202 (the fused
// streaming pass reads its halo once): up to 3.4 million cells; TE 2048^2 114
// against 133, 2560 x 2048 138 against 163, 4096 x 2048 234 against 206: 5.5
// million.  FP64: both 2048^2 377 against 399, 2560 x 2048 465 against 451: 4.3
// million; TM alone (streamed 12 sweeps deep) 2048 x 1600 132 against 147,
// 2048^2 164 against 158: 3.4 million.
// Chebyshev, 7 sweeps: FP32 1500 x 1100 70 against 93, 2048 x 1600 129 against
// 120: 2.2 million; FP64 both blocks 1024 x 1000 98 against 140, 1500 x 1100 131 against 141 in
// long calls but 176 against 158 in calls of a step, 1500 x 1400 237 against 193 so: 1.6
// million; one block 2 million.
// A step of few sweeps leaves the tiles little to win (their fronts and launches
// cost more than the streams' where the grid is large), so the limit falls with
// the sweeps m.  3 sweeps, tiles against streams in % of the streams' time: FP32 both blocks
// 1500 x 1100 93, 2048 x 1450 118; FP64 both 1500 x 1100 98, 2048^2 122, TE 2048^2 143; Chebyshev
// FP64 1024 x 1000 102, 1500 x 1100 141.  6 sweeps: FP32 both 1500 x 1400 86, 2048 x 1600 111;
// FP64 both 1500 x 1100 82, 1500 x 1400 108, TE 2048 x 1450 103, 2048 x 1600 135 (8: 94).
// By m at -3, 0, 3, 6, 8 and 12 and more, linear between, in units of 2^16 cells
// (of 700 drawn sizes, counts and calls the slower kernel is taken by more than 10 % on a dozen).
constexpr double REG_M[6] = {-3, 0, 3, 6, 8, 12};
constexpr int REG_CELLS[2][2][3][6] = {
    {{{12, 25, 36, 52, 70, 84}, {12, 25, 40, 60, 84, 84}, {12, 14, 24, 40, 46, 52}},     // FP32 TE, TM, both
     {{8, 17, 26, 42, 66, 66}, {10, 20, 28, 46, 52, 52}, {10, 14, 24, 30, 66, 66}}},     // FP64
    {{{10, 10, 24, 32, 34, 34}, {10, 10, 24, 32, 34, 34}, {10, 10, 24, 32, 34, 34}},     // Chebyshev FP32
     {{8, 10, 15, 30, 34, 34}, {8, 10, 15, 30, 34, 34}, {8, 8, 16, 22, 30, 30}}}};         // Chebyshev FP64
inline int64_t reg_cells(bool f64, int blocks, bool cheb, double m)
{
    const int *c = REG_CELLS[cheb][f64][blocks - 1];
    int i = 0;
    while (i < 4 && m > REG_M[i + 1]) i++;
    const double w = std::min(1.0, std::max(0.0, (m - REG_M[i]) / (REG_M[i + 1] - REG_M[i])));
    return (int64_t)((c[i] + w * (c[i + 1] - c[i])) * 65536.0);
}

constexpr int64_t REG_FEW = (int64_t)17 << 17;   // cells up to which calls of a few steps pay too

// A call of `steps` steps of m sweeps each on the plan p (a transposed solve,
// front = false, gains at every count: 3 sweeps, FP64, 2048^2 86 %).  filter: the
// current is filtered in a launch of its own, once per call: a step of a short
// call pays its share of it, worth about three sweeps (two of the Chebyshev
// solve; 3 sweeps, FP32 both, 1024 x 1000: 55 us against 53 in calls of a step, 29 against 32
// in calls of eight), and on the larger grids it would cost such calls what the
// tiles gain, 30 us at 2048^2 FP64.  A step without sweeps (lumped; FP64 1299 x 617, 39 us
// against 34) is told apart from one of a few.
// Grids whose short side holds little of a tile, us per step of 20 sweeps, FP32, tiles
// against streams: 46875 x 64 177 against 155, 187500 x 16 180 against 221, 375000 x 8
// 302 against 311, 750000 x 4 549 against 511, 3000000 x 1 2095 against 1495; a million
// cells, 62500 x 16 68 against 114, 125000 x 8 119 against 161, 250000 x 4 218 against
// 215, 1000000 x 1 710 against 530; 60000 cells, 15000 x 4 25 against 70; the other way
// round, 64 x 46875 188 against 299, 1 x 3000000 4587 against 14303.
inline bool reg_pays(const RegPlan &p, bool f64, int blocks, bool cheb, bool front, int64_t nx, int64_t ny, int m, int steps,
                     bool filter)
{
    using namespace reg2d;
    const double share = filter ? (cheb ? 2.0 : 3.0) / steps : 0.0;
    const int64_t most = reg_cells(f64, blocks, cheb, !front ? 1e9 : m > 0 ? m - share : -2.0 - share), n = side_of(most);
    if (p.geo < 0 || nx * ny > most || (filter && steps < 8 && nx * ny > REG_FEW)) return false;
    if (std::min(nx, ny) >= SHORT) return true;
    return tiles_win(p.us, reg_plan(f64, blocks, cheb, front, n, n, m).us, 0.55, strip_cells(nx, ny, 240, 10), most);
}

// Tolerance solves: FP32 (two tested passes) 2048 x 1600 227 against 237,
// 2048^2 286 against 286; delta form 2048 x 1450 92 %, 2048 x 1600 103 %: 3.4 million, both
// blocks in delta form 3.1.  FP64: standard form (three) 2048 x 1600 379 against
// 436, 2048^2 523 against 483, but with nine tested passes 2048 x 1450 774 against 748: 2.9
// million both blocks, 3.4 one; delta form, whose passes read and write the
// running sum too, both blocks 1500 x 1100 85 to 93 %, 1500 x 1400 104 to 114, 2048 x 1600
// 117 to 132 (by the number of passes; three to twelve): 1.8 million, one block
// 1800 x 1300 99, 2048 x 1450 104: 2.4 million.  Chebyshev: FP64 (passes of four) 1024^2
// 301 against 356, 1500 x 1100 453 against 429: 1.3 million.
inline int64_t reg_tol_cells(bool f64, int blocks, bool cheb, bool delta)
{
    if (cheb) return f64 ? (int64_t)5 << 18 : (int64_t)17 << 17;
    if (f64 && delta) return (int64_t)(blocks == 3 ? 7 : 9) << 18;
    return (int64_t)(blocks != 3 ? 13 : f64 ? 11 : delta ? 12 : 13) << 18;
}

// A tolerance solve whose tested passes have k sweeps, on its plan.  Every
// workgroup sums the norms of all before it, so the decision grows with the
// square of the tiles, about 1e-5 us per launch times the tiles squared (FP64
// Chebyshev, passes of four: 4 x 250000, 4464 tiles, 4443 us per step against
// 3232; 8 x 125000, 2232 tiles, 1671 against 1705).
inline bool reg_tol_pays(const RegPlan &p, bool f64, int blocks, bool cheb, bool delta, int64_t nx, int64_t ny, int k)
{
    using namespace reg2d;
    const int64_t most = reg_tol_cells(f64, blocks, cheb, delta), n = side_of(most);
    if (p.geo < 0 || nx * ny > most) return false;
    if (std::min(nx, ny) >= SHORT) return true;
    auto us = [&](const RegPlan &q, int64_t x, int64_t y) {
        const double t = (double)tiles(GEO[q.geo], RK_MID, (k + q.passes - 1) / q.passes, x, y);
        return q.us + 2 * q.passes * 1e-5 * t * t;
    };
    return tiles_win(us(p, nx, ny), us(reg_tol_plan(f64, blocks, cheb, n, n, k, most), n, n), 0.55,
                     strip_cells(nx, ny, 240, 10), most);
}

// Batches by register tiles against row streams, by their cells, us per step.
// FP32: 1.3 million, 14 sweeps, 72 against 107; 2.75 million, 20 sweeps, 134
// against 155; 3.3 million, 20 sweeps, 162 against 192, but with 8 sweeps 2.9
// million 83 against 87 and with 10 sweeps 98 against 97; 4.5 million, 20
// sweeps, 218 against 216.  FP64: 0.18 million, 12 sweeps, 30 against 123; 4.3
// million, 20 sweeps, 367 against 485, 8 sweeps 250 against 255; 7.2 million
// 587 against 770 and 395 against 413.
// Fewer sweeps, in % of the streams' time: FP32 1 sweep 2.2 million 105, 3 sweeps 2.2 million 99,
// 2.7 million 109; FP64 3 sweeps 1.7 million 90, 2.2 million 121, 7.2 million 125, 5 sweeps 93.
inline int64_t reg_batch_cells(bool f64, int m)
{
    if (f64) return (int64_t)(m >= 5 ? 112 : m >= 3 ? 27 : 20) << 16;
    return (int64_t)(m >= 12 ? 52 : m >= 5 ? 44 : m >= 3 ? 34 : 30) << 16;
}

inline int64_t reg_batch_tiles(int geo, int kind, int cut, int64_t nx, int64_t ny)
{
    return reg2d::tiles(reg2d::GEO[geo], kind, cut, nx, ny);
}

// geo < 0: the row streams are faster
inline RegBatchPlan reg_batch_plan(const mx_config *cfgs, int ng)
{
    using namespace reg2d;
    const bool f64 = cfgs[0].dtype == MX_F64;
    const int m = cfgs[0].sweeps;
    int64_t cells = 0;
    for (int i = 0; i < ng; i++) cells += cfgs[i].n[0] * cfgs[i].n[1];
    RegBatchPlan best{-1, 0, 0, 0};
    const int64_t most = reg_batch_cells(f64, m), side = side_of(most);
    if (cells > most) return best;
    double us = 1e29, meet = 1e29, strips = 0.0;
    const Fit *fit = FIT[0][f64 ? 5 : 2];
    // (kb_reg is built for one column per lane: without the 128 x 64 region, which
    // FP32 grids of some million cells prefer on their own)
    for (int g = 0; g < 3; g++) {
        const int kmax = std::min((GEO[g].ry - 4) / 2, 16);
        for (int n = std::max(2, (m + kmax - 1) / kmax); n <= m / 2 + 2; n++) {
            // passes of m / n sweeps, the first ones one fewer than the rest
            const int kf = m / n, ks = (m + n - 1) / n;
            auto pass = [&](int kind, int k, bool limit) {
                const int W = GEO[g].rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = GEO[g].ry - 2 * k;
                if (W < 12 || H < 4) return 1e30;
                double t = 0.0;
                for (int i = 0; i < ng && !limit; i++) t += 2.0 * tiles(GEO[g], kind, k, cfgs[i].n[0], cfgs[i].n[1]);
                if (limit) t = 2.0 * tiles(GEO[g], kind, k, side, side);
                const double c = per_cu(t);
                return fit[g].t0 + c * fit[g].load[kind] + k * (c * fit[g].s + fit[g].s0);
            };
            auto step = [&](bool limit) {
                return pass(RK_FRONT, kf, limit) + (n - 2) * pass(RK_MID, ks, limit) + pass(RK_LAST, ks, limit);
            };
            const double t = step(false);
            meet = std::min(meet, step(true));
            if (t < us) us = t, best = RegBatchPlan{g, n, kf, ks};
            if (n > 40) break;
        }
    }
    // thin grids, us per step of 20 sweeps, tiles against streams, FP32: 8 of 375000 x 1 2179
    // against 879, of 46875 x 8 312 against 236, of 23437 x 16 179 against 181; 1 million
    // cells, 31250 x 4 212 against 134, 15625 x 8 123 against 105, 7812 x 16 72 against 104; 0.2
    // million, 12500 x 2 95 against 66, 6250 x 4 56 against 62.  FP64: 46875 x 8 523 against
    // 503, 23437 x 16 317 against 394; 31250 x 4 348 against 252, 15625 x 8 199 against 215;
    // 12500 x 2 146 against 95, 6250 x 4 87 against 82
    int64_t side_min = SHORT;
    for (int i = 0; i < ng; i++) {
        strips += strip_cells(cfgs[i].n[0], cfgs[i].n[1], 224, 5);
        side_min = std::min({side_min, cfgs[i].n[0], cfgs[i].n[1]});
    }
    if (side_min < SHORT / 2 && !tiles_win(us, meet, f64 ? 0.15 : 0.37, strips, most)) best.geo = -1;
    return best;
}

}  // namespace mx
