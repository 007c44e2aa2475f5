// Particle coupling of the 2D field step (arXiv 1907.13088: the solver runs
// inside a particle-in-cell code whose force interpolation, deposition and
// push it leaves unchanged, Sec. 2; Gauss's law for E holds when the
// deposition conserves charge, Sec. 2 and Appendix A):
//   push ........ relativistic Boris scheme (Boris 1970) in E^n and
//                 B^n = B^{n-1/2} - (dt/2) curl E^n, c = 1
//   shapes ...... first-order B-spline at each component's staggered
//                 position (the lowest order of the paper's Table 1)
//   deposition .. Esirkepov's charge-conserving decomposition (Esirkepov
//                 2001), 2D with an out-of-plane current, added with
//                 floating-point atomics: in LDS when the windows of a
//                 workgroup's particles fit one tile (particles kept in cell
//                 order), then once per node into J; else directly into J
// Positions are at time level n, momenta
// u = gamma v at n - 1/2; after the call positions are at n + 1 (wrapped
// into [0, L)), momenta at n + 1/2, and J holds J^{n+1/2}.
//
// A particle moves less than one cell per axis per step: |v| < c and the
// time step obeys the CFL bound dt <= (1/dx^2 + 1/dy^2)^(-1/2) < min(dx, dy),
// so the 4 x 4 node window starting one node before the start cell covers
// both shapes.
#include <algorithm>
#include <limits>

#include "mx_internal.h"

namespace mx {
namespace {

constexpr int PT = 256;

template <typename T>
__device__ __forceinline__ T shape1(T d)
{
    d = fabs(d);
    return d < T(1) ? T(1) - d : T(0);
}

__device__ __forceinline__ int wrapn(int i, int n)
{
    i %= n;
    return i < 0 ? i + n : i;
}

// the same for indices within a few cells of [0, n): no division
__device__ __forceinline__ int wrapc(int i, int n)
{
    if (i >= 0 && i < n) return i;
    const int j = i < 0 ? i + n : i - n;
    return (j >= 0 && j < n) ? j : wrapn(i, n);
}

// q = x / d rounded as the division does, from r = 1 / d rounded: two
// remainder steps (Markstein: with r correctly rounded and the estimate
// within an ulp, the second is the correctly rounded quotient; the product
// x r alone can be 1.5 ulp off).  Five operations against the ten or so of a
// division, wherever one divisor serves several quotients.  d is finite (the
// remainder of an infinite one would be NaN); r = 0 gives x / infinity = 0.
template <typename T>
__device__ __forceinline__ T divr(T x, T d, T r)
{
    const T q = x * r;
    const T q1 = fma(fma(-q, d, x), r, q);
    return fma(fma(-q1, d, x), r, q1);
}

// x / 6: the rounded 1/6 is off by a quarter ulp at most, so the product is
// within an ulp and one remainder step rounds correctly
template <typename T>
__device__ __forceinline__ T div6(T x)
{
    const T q = x * T(1.0 / 6.0);
    return fma(fma(T(-6), q, x), T(1.0 / 6.0), q);
}

// Values of the accumulation area of the deposition in LDS: a workgroup's
// window of three components, in up to 32 copies; FP64 for both types (below)
constexpr int ACC = 4096;

// min and max of two values over the workgroup (valid in every thread)
__device__ __forceinline__ void block_minmax2(int (&v)[4], int (*sh)[4])
{
    for (int off = 32; off > 0; off >>= 1) {
        v[0] = min(v[0], __shfl_xor(v[0], off, 64));
        v[1] = max(v[1], __shfl_xor(v[1], off, 64));
        v[2] = min(v[2], __shfl_xor(v[2], off, 64));
        v[3] = max(v[3], __shfl_xor(v[3], off, 64));
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0)
        for (int q = 0; q < 4; q++) sh[w][q] = v[q];
    __syncthreads();
    for (int w2 = 0; w2 < PT / 64; w2++) {
        v[0] = min(v[0], sh[w2][0]);
        v[1] = max(v[1], sh[w2][1]);
        v[2] = min(v[2], sh[w2][2]);
        v[3] = max(v[3], sh[w2][3]);
    }
}

// Fields a particle gathers, paired by stagger so that a pair's four nodes
// are read together: {Ex, By}, {Ey, Bx}, Ez, Bz
template <typename T>
struct alignas(2 * sizeof(T)) FPair {
    T e, b;
};

// B^n = B^{n-1/2} - (dt/2) curl E^n at every node (eqs faraday_*, 2D), once
// per node instead of at the four nodes of each component of each particle
template <typename T>
__global__ __launch_bounds__(PT) void k_pic_fields(PicArgs<T> a, FPair<T> *exby, FPair<T> *eybx, T *bz)
{
    const unsigned o = blockIdx.x * PT + threadIdx.x;   // fields are below 4 GiB
    const unsigned nx = a.nx, ny = a.ny;
    if (o >= nx * ny) return;
    const unsigned j = o / nx, i = o - j * nx;
    const unsigned r = o - i + (i + 1 < nx ? i + 1 : 0), u = (j + 1 < ny ? o + nx : i);
    const T dxEz = (a.E[2][r] - a.E[2][o]) / a.dx, dyEz = (a.E[2][u] - a.E[2][o]) / a.dy;
    const T dxEy = (a.E[1][r] - a.E[1][o]) / a.dx, dyEx = (a.E[0][u] - a.E[0][o]) / a.dy;
    exby[o] = FPair<T>{a.E[0][o], a.B[1][o] - a.th * (T(0) - dxEz)};
    eybx[o] = FPair<T>{a.E[1][o], a.B[0][o] - a.th * (dyEz - T(0))};
    bz[o] = a.B[2][o] - a.th * (dxEy - dyEx);
}

// Push and deposition, `ppt` particles per thread.  PRE: the fields come from
// k_pic_fields; else (few particles per node) each particle forms its B^n.
//
// Bound: VALU issue and, before, the LDS adds.  The particles of a wavefront,
// kept in cell order, add to the same few nodes, so each workgroup sums its
// window in up to 32 copies, a lane's copy being its lane number (same-address
// adds serialise: 64 deep before, 2 now), and skips, for a whole wavefront,
// the window's outer rows and columns that none of its particles reaches.
// The sums are FP64 for both types: FP32 adds in LDS take about three cycles
// a lane on this part, FP64 adds well under one (8.4 M particles on 256 x 128
// cells in cell order, FP32: 580 us with FP32 sums, 190 with FP64 sums, 177
// with plain non-atomic ones, which lose updates), and round less.  The same
// push took 740 us with one FP32 copy, 40 adds per particle, a division for
// each quotient and B^n formed per particle; its phase space alone (40 B per
// particle) takes 67 us at the rate of a large copy.  FP64 755 -> 318 us; 8
// particles per cell on 512^2, FP32 760 -> 85 us (the window there was too
// wide for the former 32 x 32 tile, and its adds went to memory).
template <typename T, bool PRE>
__global__ __launch_bounds__(PT) void k_pic_push(PicArgs<T> a, const FPair<T> *exby, const FPair<T> *eybx, const T *bzn,
                                                 int ppt)
{
    __shared__ double acc[ACC];
    __shared__ int sh[PT / 64][4];
    const int64_t p0 = (int64_t)blockIdx.x * PT * ppt;   // the workgroup's first particle (exists)
    const int nx = a.nx, ny = a.ny, tid = threadIdx.x;
    const T dx = a.dx, dy = a.dy, dt = a.dt, rdx = T(1) / dx, rdy = T(1) / dy;
    // gamma overflows from |u| of 1.8e19 (FP64 1.3e154): the particle's velocity
    // rounds to zero
    constexpr T huge = std::numeric_limits<T>::max();
    // cells relative to the first particle's, by the shorter way around the
    // periodic box: a window may cross its edge
    const int iref = (int)floor(divr(a.x[p0], dx, rdx)), jref = (int)floor(divr(a.y[p0], dy, rdy));
    auto rel = [](int i, int ref, int n) {
        int d = (int)min(max((long long)i - ref, -(1LL << 28)), 1LL << 28);
        return d > n / 2 ? d - n : (d < -(n / 2) ? d + n : d);
    };
    int mm[4] = {0x7fffffff, -0x7fffffff, 0x7fffffff, -0x7fffffff};
    // the first round's particle, loaded ahead of the window's reduction
    T xf = T(0), yf = T(0), uf[3] = {T(0), T(0), T(0)};
    if (p0 + tid < a.np) {
        xf = a.x[p0 + tid];
        yf = a.y[p0 + tid];
        uf[0] = a.ux[p0 + tid];
        uf[1] = a.uy[p0 + tid];
        uf[2] = a.uz[p0 + tid];
    }
    for (int u = 0; u < ppt; u++) {
        const int64_t p = p0 + u * PT + tid;
        if (p >= a.np) break;
        const int di = rel((int)floor(divr(u == 0 ? xf : a.x[p], dx, rdx)), iref, nx);
        const int dj = rel((int)floor(divr(u == 0 ? yf : a.y[p], dy, rdy)), jref, ny);
        mm[0] = min(mm[0], di);
        mm[1] = max(mm[1], di);
        mm[2] = min(mm[2], dj);
        mm[3] = max(mm[3], dj);
    }
    block_minmax2(mm, sh);   // (its barrier: every thread has read the reference particle)
    const int bw = mm[1] - mm[0] + 4, bh = mm[3] - mm[2] + 4;   // the window's nodes per row, rows
    const long long area3 = 3LL * bw * bh;
    const bool in_lds = area3 <= ACC;
    int nc = 0;   // log2 of the copies
    if (in_lds) {
        while (nc < 5 && (area3 << (nc + 1)) <= ACC) nc++;
        for (int e = tid; e < ((int)area3 << nc); e += PT) acc[e] = 0.0;
        __syncthreads();
    }
    const int copy = tid & ((1 << nc) - 1);
    for (int u = 0; u < ppt; u++) {
        const int64_t p = p0 + u * PT + tid;
        const bool live = p < a.np;
        if (!__any(live)) break;
        if (u > 0 && live) {
            xf = a.x[p];
            yf = a.y[p];
            uf[0] = a.ux[p];
            uf[1] = a.uy[p];
            uf[2] = a.uz[p];
        }
        const T x0 = live ? xf : T(0), y0 = live ? yf : T(0);
        const T xi0 = divr(x0, dx, rdx), eta0 = divr(y0, dy, rdy);
        const int ic = (int)floor(xi0), jc = (int)floor(eta0);
        // linear weights at node and half-node positions: the stencil's first
        // node i0 and the weights of i0 and i0 + 1 (1 - |xi - i|, in [0, 1])
        T wx[2][2], wy[2][2];   // [half][node]
        wx[0][0] = T(1) - (xi0 - T(ic));
        wx[0][1] = T(1) + (xi0 - T(ic + 1));
        wy[0][0] = T(1) - (eta0 - T(jc));
        wy[0][1] = T(1) + (eta0 - T(jc + 1));
        const T xih = xi0 - T(0.5), etah = eta0 - T(0.5);
        const int ih = (int)floor(xih), jh = (int)floor(etah);
        wx[1][0] = T(1) - (xih - T(ih));
        wx[1][1] = T(1) + (xih - T(ih + 1));
        wy[1][0] = T(1) - (etah - T(jh));
        wy[1][1] = T(1) + (etah - T(jh + 1));
        // wrapped columns and row offsets of the 4 x 4 nodes from (ic - 1,
        // jc - 1); a half-node stencil starts at ic - 1 or ic
        unsigned cw[4], rw[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            cw[k] = (unsigned)wrapc(ic - 1 + k, nx);
            rw[k] = (unsigned)wrapc(jc - 1 + k, ny) * (unsigned)nx;
        }
        const bool hx = ih >= ic, hy = jh >= jc;
        const unsigned c0[3] = {cw[1], cw[2], cw[3]}, r0[3] = {rw[1], rw[2], rw[3]};
        const unsigned ch[3] = {hx ? cw[1] : cw[0], hx ? cw[2] : cw[1], hx ? cw[3] : cw[2]};
        const unsigned rh[3] = {hy ? rw[1] : rw[0], hy ? rw[2] : rw[1], hy ? rw[3] : rw[2]};
        T ex = T(0), ey = T(0), ez = T(0), bx = T(0), by = T(0), bz = T(0);
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const T whn = wx[1][c] * wy[0][b], wnh = wx[0][c] * wy[1][b];
                const T wnn = wx[0][c] * wy[0][b], whh = wx[1][c] * wy[1][b];
                FPair<T> f, g;
                T vz;
                if (PRE) {
                    f = exby[r0[b] + ch[c]];
                    g = eybx[rh[b] + c0[c]];
                    vz = bzn[rh[b] + ch[c]];
                } else {
                    const T *Ex = a.E[0], *Ey = a.E[1], *Ez = a.E[2];
                    const T dxEz = (Ez[r0[b] + ch[c + 1]] - Ez[r0[b] + ch[c]]) / dx;
                    const T dyEz = (Ez[rh[b + 1] + c0[c]] - Ez[rh[b] + c0[c]]) / dy;
                    const T dxEy = (Ey[rh[b] + ch[c + 1]] - Ey[rh[b] + ch[c]]) / dx;
                    const T dyEx = (Ex[rh[b + 1] + ch[c]] - Ex[rh[b] + ch[c]]) / dy;
                    f = FPair<T>{Ex[r0[b] + ch[c]], a.B[1][r0[b] + ch[c]] - a.th * (T(0) - dxEz)};
                    g = FPair<T>{Ey[rh[b] + c0[c]], a.B[0][rh[b] + c0[c]] - a.th * (dyEz - T(0))};
                    vz = a.B[2][rh[b] + ch[c]] - a.th * (dxEy - dyEx);
                }
                ex += whn * f.e;
                by += whn * f.b;
                ey += wnh * g.e;
                bx += wnh * g.b;
                ez += wnn * a.E[2][r0[b] + c0[c]];
                bz += whh * vz;
            }
        // Boris: half electric kick, rotation about B, half electric kick
        const T h = a.h;
        const T umx = uf[0] + h * ex, umy = uf[1] + h * ey, umz = uf[2] + h * ez;
        const T gm = sqrt(T(1) + umx * umx + umy * umy + umz * umz);
        const T rgm = T(1) / gm, gmf = fmin(gm, huge);
        const T tx = divr(h * bx, gmf, rgm), ty = divr(h * by, gmf, rgm), tz = divr(h * bz, gmf, rgm);
        const T upx = umx + (umy * tz - umz * ty);
        const T upy = umy + (umz * tx - umx * tz);
        const T upz = umz + (umx * ty - umy * tx);
        const T f = T(2) / (T(1) + tx * tx + ty * ty + tz * tz);
        const T sx = f * tx, sy = f * ty, sz = f * tz;
        const T uplx = umx + (upy * sz - upz * sy);
        const T uply = umy + (upz * sx - upx * sz);
        const T uplz = umz + (upx * sy - upy * sx);
        const T nux = uplx + h * ex, nuy = uply + h * ey, nuz = uplz + h * ez;
        const T g = sqrt(T(1) + nux * nux + nuy * nuy + nuz * nuz);
        const T rg = T(1) / g, gf = fmin(g, huge);
        const T x1 = x0 + divr(dt * nux, gf, rg), y1 = y0 + divr(dt * nuy, gf, rg);
        const T vz = divr(nuz, gf, rg);
        // Esirkepov: shapes of the start and end positions on the window of
        // nodes ic - 1 .. ic + 2, jc - 1 .. jc + 2 (the start position's
        // outer weights are zero)
        const T xi1 = divr(x1, dx, rdx), eta1 = divr(y1, dy, rdy);
        const T sx0[4] = {T(0), wx[0][0], wx[0][1], T(0)}, sy0[4] = {T(0), wy[0][0], wy[0][1], T(0)};
        T sx1[4], sy1[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            sx1[k] = shape1(xi1 - T(ic - 1 + k));
            sy1[k] = shape1(eta1 - T(jc - 1 + k));
        }
        // window columns and rows some particle of the wavefront reaches
        const bool xl = __any(live && sx1[0] != T(0)), xr = __any(live && sx1[3] != T(0));
        const bool yl = __any(live && sy1[0] != T(0)), yr = __any(live && sy1[3] != T(0));
        if (live) {
            a.x[p] = x1 >= a.Lx ? x1 - a.Lx : (x1 < T(0) ? x1 + a.Lx : x1);
            a.y[p] = y1 >= a.Ly ? y1 - a.Ly : (y1 < T(0) ? y1 + a.Ly : y1);
            a.ux[p] = nux;
            a.uy[p] = nuy;
            a.uz[p] = nuz;
        }
        const int di = rel(ic, iref, nx) - mm[0], dj = rel(jc, jref, ny) - mm[2];
        auto add = [&](int comp, int k, int l, T v) {
            if (in_lds) {
                unsafeAtomicAdd(&acc[(((comp * bh + dj + l) * bw + di + k) << nc) + copy], (double)v);
            } else if (v != T(0)) {
                unsafeAtomicAdd(&a.J[comp][(size_t)wrapc(jc - 1 + l, ny) * nx + wrapc(ic - 1 + k, nx)], v);
            }
        };
        if (live) {
#pragma unroll
            for (int l = 0; l < 4; l++) {
                if ((l == 0 && !yl) || (l == 3 && !yr)) continue;
                T run = T(0);   // sum of W_x over the window's nodes up to k
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    if ((k == 0 && !xl) || (k == 2 && !xr)) continue;
                    run += T(0.5) * (sx1[k] - sx0[k]) * (sy0[l] + sy1[l]);
                    add(0, k, l, a.cx * run);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if ((k == 0 && !xl) || (k == 3 && !xr)) continue;
                T run = T(0);   // sum of W_y over the window's nodes up to l
#pragma unroll
                for (int l = 0; l < 3; l++) {
                    if ((l == 0 && !yl) || (l == 2 && !yr)) continue;
                    run += T(0.5) * (sy1[l] - sy0[l]) * (sx0[k] + sx1[k]);
                    add(1, k, l, a.cy * run);
                }
            }
#pragma unroll
            for (int l = 0; l < 4; l++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    if ((l == 0 && !yl) || (l == 3 && !yr) || (k == 0 && !xl) || (k == 3 && !xr)) continue;
                    const T wz = div6(T(2) * sx0[k] * sy0[l] + sx1[k] * sy0[l] + sx0[k] * sy1[l] + T(2) * sx1[k] * sy1[l]);
                    add(2, k, l, a.cz * vz * wz);
                }
        }
    }
    if (in_lds) {
        __syncthreads();
        for (int e = tid; e < (int)area3; e += PT) {
            double s = 0.0;
            for (int q = 0; q < (1 << nc); q++) s += acc[(e << nc) + ((q + tid) & ((1 << nc) - 1))];   // spread over the banks
            const T v = (T)s;
            if (v == T(0)) continue;
            const int c = e / (bw * bh), r = e - c * bw * bh, l = r / bw, k = r - l * bw;
            unsafeAtomicAdd(&a.J[c][(size_t)wrapn(jref + mm[2] - 1 + l, ny) * nx + wrapn(iref + mm[0] - 1 + k, nx)], v);
        }
    }
}

// rho at the nodes += q w / (dx dy) S(x/dx - i) S(y/dy - j)
template <typename T>
__global__ __launch_bounds__(PT) void k_pic_charge(int64_t np, int nx, int ny, T dx, T dy, T cq, const T *x,
                                                   const T *y, T *rho)
{
    const int64_t p = (int64_t)blockIdx.x * PT + threadIdx.x;
    if (p >= np) return;
    const T xi = x[p] / dx, eta = y[p] / dy;
    const int i0 = (int)floor(xi), j0 = (int)floor(eta);
    for (int b = 0; b < 2; b++)
        for (int c = 0; c < 2; c++) {
            const T v = cq * shape1(xi - T(i0 + c)) * shape1(eta - T(j0 + b));
            if (v != T(0)) unsafeAtomicAdd(&rho[(size_t)wrapn(j0 + b, ny) * nx + wrapn(i0 + c, nx)], v);
        }
}

template <typename T>
__global__ __launch_bounds__(PT) void k_fill0(int64_t n, T *a, T *b, T *c)
{
    const int64_t i = (int64_t)blockIdx.x * PT + threadIdx.x;
    if (i >= n) return;
    a[i] = T(0);
    if (b) b[i] = T(0);
    if (c) c[i] = T(0);
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + PT - 1) / PT); }

}  // namespace

template <typename T>
hipError_t launch_pic_push(const PicArgs<T> &a, bool zero_j, void *scratch, hipStream_t s)
{
    const int64_t ncell = (int64_t)a.nx * a.ny;
    if (zero_j && ncell > 0)
        hipLaunchKernelGGL((k_fill0<T>), dim3(blocks_for(ncell)), dim3(PT), 0, s, ncell, a.J[0], a.J[1], a.J[2]);
    if (a.np <= 0) return hipGetLastError();
    // up to four particles per thread while 2048 workgroups remain: a
    // workgroup's window, its clearing and its adds to J serve more of them
    // (fewer where they would spread over more cells than the window holds)
    const int ppt = (int)std::max<int64_t>(1, std::min<int64_t>({4, a.np / (2048 * PT), a.np / (2 * ncell)}));
    const unsigned nb = (unsigned)((a.np + (int64_t)PT * ppt - 1) / ((int64_t)PT * ppt));
    FPair<T> *exby = (FPair<T> *)scratch, *eybx = exby + ncell;
    T *bz = (T *)(eybx + ncell);
    // the node fields pay off once they serve several particles per node and
    // the push is long against one more launch (us, without and with them: 256 x 128,
    // 200000 particles, FP32 in random order 132 and 123, by rows 113 and 100, in cell order
    // 27 and 27; 42000 in cell order 21 and 26; 2048^2, a million FP32 in cell order 296
    // and 330, at random 700 and 537)
    if (a.np >= std::max<int64_t>(ncell / 2, 1 << 17)) {
        hipLaunchKernelGGL((k_pic_fields<T>), dim3(blocks_for(ncell)), dim3(PT), 0, s, a, exby, eybx, bz);
        hipLaunchKernelGGL((k_pic_push<T, true>), dim3(nb), dim3(PT), 0, s, a, exby, eybx, bz, ppt);
    } else {
        hipLaunchKernelGGL((k_pic_push<T, false>), dim3(nb), dim3(PT), 0, s, a, nullptr, nullptr, nullptr, ppt);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pic_charge(int64_t np, int nx, int ny, T dx, T dy, T cq, const T *x, const T *y, T *rho,
                             bool zero_rho, hipStream_t s)
{
    const int64_t ncell = (int64_t)nx * ny;
    if (zero_rho && ncell > 0)
        hipLaunchKernelGGL((k_fill0<T>), dim3(blocks_for(ncell)), dim3(PT), 0, s, ncell, rho, (T *)nullptr,
                           (T *)nullptr);
    if (np > 0) hipLaunchKernelGGL((k_pic_charge<T>), dim3(blocks_for(np)), dim3(PT), 0, s, np, nx, ny, dx, dy, cq, x, y, rho);
    return hipGetLastError();
}

template hipError_t launch_pic_push<float>(const PicArgs<float> &, bool, void *, hipStream_t);
template hipError_t launch_pic_push<double>(const PicArgs<double> &, bool, void *, hipStream_t);
template hipError_t launch_pic_charge<float>(int64_t, int, int, float, float, float, const float *, const float *,
                                             float *, bool, hipStream_t);
template hipError_t launch_pic_charge<double>(int64_t, int, int, double, double, double, const double *,
                                              const double *, double *, bool, hipStream_t);

}  // namespace mx
