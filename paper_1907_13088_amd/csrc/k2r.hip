// Register-tile passes of the 2D step: choice of tile and depth, dispatch
// (the kernels are instantiated in k2r_{f32,f64}_{std,tol,cheb,ctol}.hip), and the
// filter of the current that runs once per call ahead of them.
#include <algorithm>
#include <cmath>

#include "k2r_impl.h"

namespace mx {
namespace reg2d {

template <typename T, int FORM, bool TOL>
hipError_t launch(const Coef<T> &c, int mask, int geo, int kind, const RegArgs<T> &a, hipStream_t s, int *npart);
#define MX_REG_EXTERN(T, F, TOL) \
    extern template hipError_t launch<T, F, TOL>(const Coef<T> &, int, int, int, const RegArgs<T> &, hipStream_t, int *);
#define MX_REG_EXTERN_T(T)                                                                                             \
    MX_REG_EXTERN(T, FM_STD, false) MX_REG_EXTERN(T, FM_CHEB, false) MX_REG_EXTERN(T, FM_STD, true)                     \
    MX_REG_EXTERN(T, FM_DELTA, true) MX_REG_EXTERN(T, FM_CHEB, true)
MX_REG_EXTERN_T(float)
MX_REG_EXTERN_T(double)
#undef MX_REG_EXTERN_T
#undef MX_REG_EXTERN

// Tile geometries: columns and rows of the region.  Two neighbouring columns
// per lane (FP32) halve the lane shifts and widen the region; in FP64 they
// leave a CU one workgroup, and nothing hides its loads (1500 x 1100, 8
// sweeps, TE 72 against 41 us).
struct Geo {
    int rx, ry;
};
constexpr Geo GEO[4] = {{64, 32}, {64, 32}, {64, 64}, {128, 64}};

// Time of a pass (us) with c workgroups per CU: t0 + c load[kind] + k (c s + s0),
// fitted to sweeps over grids from 128^2 to 2048^2, depths 0 to 14, every
// geometry, each block alone and both in one launch (relative rms 5 to 20 %;
// the choice it makes is within 3 % of the best measured one on average, 35 %
// at worst).  By form (standard and delta, Chebyshev), type and blocks,
// geometry.
struct Fit {
    double t0, load[3], s, s0;
};
constexpr Fit FIT[2][6][4] = {
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
double per_cu(double n) { return n <= 1024 ? std::ceil(n / 256) : n / 256 + 0.5; }

// workgroups per block of a pass
int64_t tiles(const Geo &g, int kind, int k, int64_t nx, int64_t ny)
{
    const int W = g.rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = g.ry - 2 * k;
    return ((nx + W - 1) / W) * ((ny + H - 1) / H);
}

double pass_us(const Fit &f, const Geo &g, int blocks, int kind, int k, int64_t nx, int64_t ny)
{
    const int W = g.rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = g.ry - 2 * k;
    if (W < 12 || H < 4) return 1e30;
    const double c = per_cu((double)tiles(g, kind, k, nx, ny) * (blocks == 3 ? 2 : 1));
    return f.t0 + c * f.load[kind] + k * (c * f.s + f.s0);
}

// columns the block of threads filters, and rows per thread block
constexpr int FX = 64, FYR = 16;

// p passes of (1,2,1)/4 along x and y of one component per blockIdx.y: x by
// the (2p + 1)-tap binomial, y by p cascaded three-tap passes, the
// operations of the row-streaming front in its order
template <typename T, int P>
__global__ __launch_bounds__(256) void k2_filter(int nx, int ny, int ntx, const T *s0, const T *s1, const T *s2, T *d0, T *d1, T *d2,
                                                 const int *stall, int epoch)
{
    if (stall != nullptr && *stall == epoch) return;
    constexpr int RXJ = FX + 2 * P, RYJ = FYR + 2 * P;
    __shared__ T raw[RYJ][RXJ];
    __shared__ T fx[RYJ][FX];
    const T *src = blockIdx.y == 0 ? s0 : (blockIdx.y == 1 ? s1 : s2);
    T *dst = blockIdx.y == 0 ? d0 : (blockIdx.y == 1 ? d1 : d2);
    if (dst == nullptr) return;   // a component of a block that is not stepped (the whole workgroup)
    const int X0 = (int)(blockIdx.x % ntx) * FX, Y0 = (int)(blockIdx.x / ntx) * FYR;
    for (int e = threadIdx.x; e < RYJ * RXJ; e += 256) {
        const int y = e / RXJ, x = e % RXJ;
        raw[y][x] = src[(size_t)front2d::wrapi(Y0 - P + y, ny) * nx + front2d::wrapi(X0 - P + x, nx)];
    }
    __syncthreads();
    const int x = threadIdx.x & 63;
    for (int y = threadIdx.x >> 6; y < RYJ; y += 4) {
        T v = T(0);
#pragma unroll
        for (int k = -P; k <= P; k++) v = fma(T(front2d::binom<P>(k + P)), raw[y][x + P + k], v);
        fx[y][x] = v;
    }
    __syncthreads();
    if (X0 + x >= nx) return;
    for (int y = threadIdx.x >> 6; y < FYR && Y0 + y < ny; y += 4) {
        T w[2 * P + 1];
#pragma unroll
        for (int i = 0; i <= 2 * P; i++) w[i] = fx[y + i][x];
#pragma unroll
        for (int r = 1; r <= P; r++)
#pragma unroll
            for (int i = 0; i + 2 * r <= 2 * P; i++) w[i] = T(0.25) * fma(T(2), w[i + 1], w[i] + w[i + 2]);
        dst[(size_t)(Y0 + y) * nx + X0 + x] = w[0];
    }
}

// E += dE of the blocks (those with sweeps) once all have finished, the
// step's record, and B handed back; four cells per thread
constexpr int FNT = 256, FPER = 4;
template <typename T>
__global__ __launch_bounds__(FNT) void k2_reg_finish(RegFinish<T> f)
{
    __shared__ RegTolBlock sb[2];
    if (*f.tol.stall == f.tol.epoch) return;
    const int w = threadIdx.x >> 6;
    if (w < 2 && (f.blocks & (1 << w))) {
        const RegTolBlock s = reg_tol_decide(f.tol, w);
        if ((threadIdx.x & 63) == 0) {
            sb[w] = s;
            if (blockIdx.x == 0) f.tol.state[f.tol.par * 2 + w] = s;
        }
    }
    __syncthreads();
    SmallStat st{};
    st.finished = 1;
    const T *inc[3] = {nullptr, nullptr, nullptr};
    const bool w0 = blockIdx.x == 0 && threadIdx.x == 0;
#pragma unroll
    for (int b = 0; b < 2; b++) {
        if (!(f.blocks & (1 << b))) continue;
        const RegTolBlock s = sb[b];
        st.done[b] = s.done;
        st.conv[b] = s.conv;
        st.resid[b] = s.resid;
        st.rhsn[b] = s.rhsn;
        st.nonfinite |= s.nonfinite;
        if (!s.skip && s.done < f.target) st.finished = 0;
#pragma unroll
        for (int q = 0; q < 3; q++)
            if ((q == 2) == (b == 1) && s.done > 0) inc[q] = s.last == 1 ? f.inc[1][q] : f.inc[0][q];
    }
    if (w0) {
        *f.rec = st;
        if (!st.finished || st.nonfinite) *f.stall = f.tol.epoch;
    }
    if (!st.finished || st.nonfinite) return;
    const int64_t i0 = (int64_t)blockIdx.x * (FNT * FPER) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < FPER; u++) {
        const int64_t i = i0 + u * FNT;
        if (i >= f.n) return;
#pragma unroll
        for (int q = 0; q < 3; q++) {
            if (inc[q]) f.E[q][i] += ((gptr<const T>)inc[q])[i];
            if (f.Bd[q]) f.Bd[q][i] = f.Bs[q][i];
        }
    }
}

}  // namespace reg2d

RegPlan reg_plan(bool f64, int blocks, bool cheb, bool front, int64_t nx, int64_t ny, int m)
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

// Batches by register tiles against row streams, by their cells, us per step.
// FP32: 1.3 million, 14 sweeps, 72 against 107; 2.75 million, 20 sweeps, 134
// against 155; 3.3 million, 20 sweeps, 162 against 192, but with 8 sweeps 2.9
// million 83 against 87 and with 10 sweeps 98 against 97; 4.5 million, 20
// sweeps, 218 against 216.  FP64: 0.18 million, 12 sweeps, 30 against 123; 4.3
// million, 20 sweeps, 367 against 485, 8 sweeps 250 against 255; 7.2 million
// 587 against 770 and 395 against 413.
static bool reg_batch_pays(bool f64, int m, int64_t cells)
{
    return cells <= (f64 ? (int64_t)14 << 19 : (int64_t)(m >= 12 ? 13 : 11) << 18);
}

int64_t reg_batch_tiles(int geo, int kind, int cut, int64_t nx, int64_t ny)
{
    return reg2d::tiles(reg2d::GEO[geo], kind, cut, nx, ny);
}

RegBatchPlan reg_batch_plan(const mx_config *cfgs, int ng)
{
    using namespace reg2d;
    const bool f64 = cfgs[0].dtype == MX_F64;
    const int m = cfgs[0].sweeps;
    int64_t cells = 0;
    for (int i = 0; i < ng; i++) cells += cfgs[i].n[0] * cfgs[i].n[1];
    RegBatchPlan best{-1, 0, 0, 0};
    if (!reg_batch_pays(f64, m, cells)) return best;
    double us = 1e29;
    const Fit *fit = FIT[0][f64 ? 5 : 2];
    for (int g = 0; g < 3; g++) {
        const int kmax = std::min((GEO[g].ry - 4) / 2, 16);
        for (int n = std::max(2, (m + kmax - 1) / kmax); n <= m / 2 + 2; n++) {
            // passes of m / n sweeps, the first ones one fewer than the rest
            const int kf = m / n, ks = (m + n - 1) / n;
            auto pass = [&](int kind, int k) {
                const int W = GEO[g].rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = GEO[g].ry - 2 * k;
                if (W < 12 || H < 4) return 1e30;
                double t = 0.0;
                for (int i = 0; i < ng; i++) t += 2.0 * tiles(GEO[g], kind, k, cfgs[i].n[0], cfgs[i].n[1]);
                const double c = per_cu(t);
                return fit[g].t0 + c * fit[g].load[kind] + k * (c * fit[g].s + fit[g].s0);
            };
            const double t = pass(RK_FRONT, kf) + (n - 2) * pass(RK_MID, ks) + pass(RK_LAST, ks);
            if (t < us) us = t, best = RegBatchPlan{g, n, kf, ks};
            if (n > 40) break;
        }
    }
    return best;
}

RegPlan reg_tol_plan(bool f64, int blocks, bool cheb, int64_t nx, int64_t ny, int k, int64_t stride)
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
// Tolerance solves: FP32 (two tested passes) 2048 x 1600 227 against 237,
// 2048^2 286 against 286; FP64 (three) 379 against 436, 523 against 483: 3.4
// million.
// Chebyshev, 7 sweeps: FP32 1500 x 1100 70 against 93, 2048 x 1600 129 against
// 120; FP64 131 against 141, 244 against 241: 2.2 million; its FP64 tolerance
// solves (passes of four) 1024^2 301 against 356, 1500 x 1100 453 against 429:
// 1.3 million.
bool reg_pays(bool f64, int blocks, bool tol, bool cheb, int64_t nx, int64_t ny)
{
    int64_t most = (int64_t)13 << 18;
    if (cheb) most = tol && f64 ? (int64_t)5 << 18 : (int64_t)17 << 17;
    else if (!tol && f64 && blocks != 2) most = (int64_t)33 << 17;
    else if (!tol && !f64 && blocks != 3) most = (int64_t)21 << 18;
    return nx * ny <= most;
}

template <typename T>
hipError_t launch_reg(const Coef<T> &c, int blocks, int geo, int kind, int form, bool tol, const RegArgs<T> &a, hipStream_t s,
                      int *npart)
{
    using namespace reg2d;
    if (form == FM_STD) return tol ? launch<T, FM_STD, true>(c, blocks, geo, kind, a, s, npart) : launch<T, FM_STD, false>(c, blocks, geo, kind, a, s, npart);
    if (form == FM_CHEB) return tol ? launch<T, FM_CHEB, true>(c, blocks, geo, kind, a, s, npart) : launch<T, FM_CHEB, false>(c, blocks, geo, kind, a, s, npart);
    return tol ? launch<T, FM_DELTA, true>(c, blocks, geo, kind, a, s, npart) : hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_reg_finish(const RegFinish<T> &f, hipStream_t s)
{
    using namespace reg2d;
    const int64_t nb = (f.n + FNT * FPER - 1) / (FNT * FPER);
    hipLaunchKernelGGL((k2_reg_finish<T>), dim3((unsigned)nb), dim3(FNT), 0, s, f);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_filter2d(const Coef<T> &c, int passes, int mask, const T *const J0[3], T *const out[3], const int *stall,
                           int epoch, hipStream_t s)
{
    using namespace reg2d;
    const int ntx = (c.nx + FX - 1) / FX;
    const dim3 grid(ntx * ((c.ny + FYR - 1) / FYR), 3);
    T *d[3];
    for (int q = 0; q < 3; q++) d[q] = (mask >> q) & 1 ? out[q] : nullptr;
    switch (passes) {
    case 1: hipLaunchKernelGGL((k2_filter<T, 1>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2], stall, epoch); break;
    case 2: hipLaunchKernelGGL((k2_filter<T, 2>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2], stall, epoch); break;
    case 3: hipLaunchKernelGGL((k2_filter<T, 3>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2], stall, epoch); break;
    case 4: hipLaunchKernelGGL((k2_filter<T, 4>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2], stall, epoch); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define MX_REG_INST(T)                                                                                                          \
    template hipError_t launch_reg<T>(const Coef<T> &, int, int, int, int, bool, const RegArgs<T> &, hipStream_t, int *); \
    template hipError_t launch_reg_finish<T>(const RegFinish<T> &, hipStream_t);
MX_REG_INST(float)
MX_REG_INST(double)
#undef MX_REG_INST
template hipError_t launch_filter2d<float>(const Coef<float> &, int, int, const float *const[3], float *const[3], const int *, int, hipStream_t);
template hipError_t launch_filter2d<double>(const Coef<double> &, int, int, const double *const[3], double *const[3], const int *, int, hipStream_t);

}  // namespace mx
