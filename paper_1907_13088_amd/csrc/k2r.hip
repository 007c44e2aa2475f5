// Register-tile passes of the 2D step: dispatch (the kernels are instantiated
// in k2r_{f32,f64}_{std,tol,cheb,ctol}.hip, tile and depth chosen in plan2r.h),
// and the filter of the current that runs once per call ahead of them.
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
