// Register-tile passes of the 2D step: choice of tile and depth, dispatch
// (the kernels are instantiated in k2r_{f32,f64}_{te,tm,all}.hip), and the
// filter of the current that runs once per call ahead of them.
#include <algorithm>
#include <cmath>

#include "k2f_impl.h"
#include "mx_internal.h"

namespace mx {
namespace reg2d {

template <typename T, int BLK>
hipError_t launch(const Coef<T> &c, int geo, int kind, const RegArgs<T> &a, hipStream_t s);
#define MX_REG_EXTERN(T)                                                                             \
    extern template hipError_t launch<T, 1>(const Coef<T> &, int, int, const RegArgs<T> &, hipStream_t); \
    extern template hipError_t launch<T, 2>(const Coef<T> &, int, int, const RegArgs<T> &, hipStream_t); \
    extern template hipError_t launch<T, 3>(const Coef<T> &, int, int, const RegArgs<T> &, hipStream_t);
MX_REG_EXTERN(float)
MX_REG_EXTERN(double)
#undef MX_REG_EXTERN

// Tile geometries: columns and rows of the region.  Two neighbouring columns
// per lane halve the lane shifts and widen the region, at registers that
// leave both blocks together no room.
struct Geo {
    int rx, ry;
};
constexpr Geo GEO[4] = {{64, 32}, {64, 32}, {64, 64}, {128, 64}};

// Time of a pass (us) with c workgroups per CU: t0 + c load[kind] + k (c s + s0),
// fitted to sweeps over grids from 128^2 to 4096 x 2048, depths 0 to 14 and
// every geometry (relative rms 6 to 14 %; the choice it makes is within 6 %
// of the best measured one on most grids).  Rows: FP32 TE, TM, both, FP64
// the same; columns: geometry.
struct Fit {
    double t0, load[3], s, s0;
};
constexpr Fit FIT[6][4] = {
        {{1.31, {1.92, 1.50, 1.97}, 0.083, 0.214},
         {1.70, {1.79, 1.23, 1.76}, 0.022, 0.271},
         {0.00, {4.01, 3.12, 4.14}, 0.123, 0.368},
         {1.24, {9.16, 6.75, 8.65}, 0.094, 0.629}},   // F32 TE
        {{1.58, {1.62, 1.00, 1.14}, 0.113, 0.151},
         {1.88, {1.41, 0.70, 0.87}, 0.061, 0.181},
         {1.01, {3.06, 1.71, 2.08}, 0.176, 0.224},
         {1.58, {7.83, 3.42, 4.21}, 0.176, 0.400}},   // F32 TM
        {{0.62, {3.70, 2.40, 3.27}, 0.113, 0.357},
         {0.87, {3.47, 2.24, 3.21}, 0.028, 0.491},
         {0.00, {6.41, 3.90, 5.63}, 0.376, 0.392}},   // F32 both
        {{0.74, {3.81, 3.12, 3.81}, 0.023, 0.382},
         {1.24, {3.45, 2.68, 3.44}, 0.000, 0.396},
         {0.00, {7.15, 5.60, 6.84}, 0.182, 0.440},
         {0.00, {13.36, 9.45, 11.88}, 1.001, 0.000}},   // F64 TE
        {{1.27, {2.93, 1.49, 1.80}, 0.135, 0.251},
         {1.55, {2.74, 1.24, 1.56}, 0.065, 0.313},
         {0.28, {6.87, 2.92, 3.47}, 0.265, 0.281},
         {0.00, {11.83, 5.62, 6.54}, 0.853, 0.000}},   // F64 TM
        {{0.00, {8.61, 4.50, 5.54}, 0.179, 0.416},
         {0.00, {7.16, 4.74, 6.54}, 0.053, 0.462},
         {0.00, {12.09, 7.46, 9.70}, 1.114, 0.000}},   // F64 both
};

// workgroups per CU of a launch of n: whole ones while they are few
double per_cu(double n) { return n <= 1024 ? std::ceil(n / 256) : n / 256 + 0.5; }

double pass_us(const Fit &f, const Geo &g, int kind, int k, int64_t nx, int64_t ny)
{
    const int W = g.rx - 2 * k - (kind == RK_FRONT ? 3 : 0), H = g.ry - 2 * k;
    if (W < 12 || H < 4) return 1e30;
    const double c = per_cu((double)((nx + W - 1) / W) * (double)((ny + H - 1) / H));
    return f.t0 + c * f.load[kind] + k * (c * f.s + f.s0);
}

// columns the block of threads filters, and rows per thread block
constexpr int FX = 64, FYR = 16;

// p passes of (1,2,1)/4 along x and y of one component per blockIdx.y: x by
// the (2p + 1)-tap binomial, y by p cascaded three-tap passes, the
// operations of the row-streaming front in its order
template <typename T, int P>
__global__ __launch_bounds__(256) void k2_filter(int nx, int ny, int ntx, const T *s0, const T *s1, const T *s2, T *d0, T *d1, T *d2)
{
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

}  // namespace reg2d

RegPlan reg_plan(bool f64, int blocks, bool front, int64_t nx, int64_t ny, int m)
{
    using namespace reg2d;
    RegPlan best{-1, 0, 1e29};
    const Fit *fit = FIT[(f64 ? 3 : 0) + blocks - 1];
    for (int g = 0; g < (blocks == 3 ? 3 : 4); g++) {
        // FP64 workgroups of 128 columns hold a CU alone, so no second one
        // hides their loads: 1500 x 1100, 8 sweeps, TE 72 against 41 us on
        // 64 x 32 regions; where a CU has one workgroup only (1024^2, 20
        // sweeps: 53 against 55) the wider region's smaller halo wins
        if (f64 && g == 3 && nx * ny > (int64_t)5 << 18) continue;
        const int kmax = (GEO[g].ry - 4) / 2;
        const int n0 = std::max(front ? 2 : 1, (m + kmax - 1) / kmax);
        for (int n = n0; n <= n0 + 6; n++) {
            double t = 0.0;
            for (int i = 0, rem = m; i < n; i++) {
                const int k = rem / (n - i);
                const int kind = front && i == 0 ? RK_FRONT : (front && i == n - 1 ? RK_LAST : RK_MID);
                t += pass_us(fit[g], GEO[g], kind, k, nx, ny);
                rem -= k;
            }
            if (t < best.us) best = RegPlan{g, n, t};
        }
    }
    return best;
}

// Register tiles against row streams, us per step with current and filter at
// 20 and at 8 sweeps.  FP32, both blocks: 1024^2 61 and 38 against 130 and
// 67, 2048 x 1600 153 and 96 against 168 and 96, 2048^2 213 and 141 against
// 201 and 113 (the fused streaming pass needs no second read of its halo):
// up to 3.4 million cells.  One block, or FP64 (which streams each block on
// its own): 2048^2 FP32 TE 112 and 70 against 133 and 76, FP64 both 388 and
// 259 against 402 and 275, 2160^2 FP64 425 and 286 against 423 and 273: up to
// 4.3 million.
bool reg_pays(bool f64, int blocks, int64_t nx, int64_t ny)
{
    return nx * ny <= (!f64 && blocks == 3 ? (int64_t)13 << 18 : (int64_t)33 << 17);
}

template <typename T>
hipError_t launch_reg(const Coef<T> &c, int blocks, int geo, int kind, const RegArgs<T> &a, hipStream_t s)
{
    if (blocks == 1) return reg2d::launch<T, 1>(c, geo, kind, a, s);
    if (blocks == 2) return reg2d::launch<T, 2>(c, geo, kind, a, s);
    if (blocks == 3) return reg2d::launch<T, 3>(c, geo, kind, a, s);
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_filter2d(const Coef<T> &c, int passes, int mask, const T *const J0[3], T *const out[3], hipStream_t s)
{
    using namespace reg2d;
    const int ntx = (c.nx + FX - 1) / FX;
    const dim3 grid(ntx * ((c.ny + FYR - 1) / FYR), 3);
    T *d[3];
    for (int q = 0; q < 3; q++) d[q] = (mask >> q) & 1 ? out[q] : nullptr;
    switch (passes) {
    case 1: hipLaunchKernelGGL((k2_filter<T, 1>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2]); break;
    case 2: hipLaunchKernelGGL((k2_filter<T, 2>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2]); break;
    case 3: hipLaunchKernelGGL((k2_filter<T, 3>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2]); break;
    case 4: hipLaunchKernelGGL((k2_filter<T, 4>), grid, dim3(256), 0, s, c.nx, c.ny, ntx, J0[0], J0[1], J0[2], d[0], d[1], d[2]); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template hipError_t launch_reg<float>(const Coef<float> &, int, int, int, const RegArgs<float> &, hipStream_t);
template hipError_t launch_reg<double>(const Coef<double> &, int, int, int, const RegArgs<double> &, hipStream_t);
template hipError_t launch_filter2d<float>(const Coef<float> &, int, int, const float *const[3], float *const[3], hipStream_t);
template hipError_t launch_filter2d<double>(const Coef<double> &, int, int, const double *const[3], double *const[3], hipStream_t);

}  // namespace mx
