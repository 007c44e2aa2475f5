#pragma once
// Register-tile passes of the 2D field step (arXiv 1907.13088, Sec. 2.2.2
// and Alg 1) for grids too small to fill the GPU with row streams: the front
// (Faraday update of B, auxiliary increment dE'), k fused sweeps
// x_l = dE' + A x_(l-1) of Alg 1 and the E increment, each optional, so that
// one launch runs a whole step or a part of it.
//
// A workgroup of NW wavefronts owns a region of RX x RY cells (RX = 64 CPL
// columns, CPL neighbouring columns per lane; RY = NW R rows, R rows per
// wavefront) and holds the iterate and dE' of every cell in registers.  A
// sweep works through a lane's R rows in order; neighbour columns come by
// whole-wavefront DPP lane shifts, neighbour rows from the lane's own
// registers, and only the first and last row of each wavefront go through
// double-buffered LDS rows: one barrier per sweep, however many rows a
// workgroup has, where a row stream pays one per row.  The valid part of the
// region shrinks by one cell per side and sweep, so a pass of k sweeps
// writes (RX - 2k) x (RY - 2k) cells (with the front: three columns fewer);
// k is a run-time argument.  Values outside the valid part feed only cells
// outside the next sweep's valid part.
//
// Every value is formed by the operations of the row-streaming and LDS-tile
// kernels in the same order, so all schedules give bitwise equal fields.
//
// Bound: VALU issue (FP32, both blocks, four rows per wavefront: 27 VALU and
// 1.5 LDS instructions per cell and sweep against the row stream's 21 and
// 3; 1024^2, 441 regions of 64 x 64: 1.2 us per sweep, the issue limit of
// 1.8 M region cells), and below that the latency of a sweep (0.25 to 0.5
// us) and the 3 to 6 us of a launch with its loads and stores.  What it
// replaced was bound by latency: the LDS-tile kernel ran 128^2 on 32
// workgroups, a row stream of 1024^2 has one wavefront per SIMD and pays
// about 1 us per row.  Per step with 20 sweeps: 128^2 FP64 TM 51 -> 18 us (one
// step per call), 700 x 300 FP32 p = 3 103 -> 26 us, 1024^2 FP64 p = 3 307 ->
// 108 us.
#include <algorithm>

#include "k2f_impl.h"
#include "mx_internal.h"
#include "stencil2d.h"

namespace mx {
namespace reg2d {

using front2d::avg6;

// value of the neighbouring lane (zero past the wavefront's edge)
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
template <typename T>
__device__ __forceinline__ T from_left(T v) { return dpp<0x138>(v); }    // wave_shr:1, lane - 1
template <typename T>
__device__ __forceinline__ T from_right(T v) { return dpp<0x130>(v); }   // wave_shl:1, lane + 1

// value of column c - 1 / c + 1 of a lane's row of CPL columns
template <typename T, int CPL>
__device__ __forceinline__ T left_of(const T (&v)[CPL], int c) { return c > 0 ? v[c > 0 ? c - 1 : 0] : from_left(v[CPL - 1]); }
template <typename T, int CPL>
__device__ __forceinline__ T right_of(const T (&v)[CPL], int c)
{
    return c + 1 < CPL ? v[c + 1 < CPL ? c + 1 : 0] : from_right(v[0]);
}

template <int BLK> constexpr int ncomp() { return BLK == 3 ? 3 : BLK == 1 ? 2 : 1; }

// CPL values of one lane, one LDS access
template <typename T, int CPL>
struct alignas(CPL * sizeof(T)) Cols {
    T v[CPL];
};

// LDS rows a wavefront publishes per sweep: its first row (Ex, Ez: the next
// row of the wavefront before it) and its last row (Ex, Ey, Ez: the previous
// row of the wavefront after it)
template <int BLK> constexpr int up_rows() { return BLK == 3 ? 2 : 1; }
template <int BLK> constexpr int dn_rows() { return ncomp<BLK>(); }
template <typename T, int BLK, int CPL, int NW>
constexpr size_t lds_bytes() { return sizeof(T) * 2 * NW * (up_rows<BLK>() + dn_rows<BLK>()) * 64 * CPL; }

// quantities of one row that its own update and the neighbouring rows' use
template <typename T, int CPL>
struct Row {
    T ex[CPL], wg[CPL], h[CPL], ly[CPL];   // Ex, Ey(i+1) - Ey(i), Ex(i) - Ex(i-1), Dxx Ey
    T ez[CPL], lx[CPL];                    // Ez, Dxx Ez
};

template <typename T, int BLK, int CPL, int R, int NW>
struct Tile {
    static constexpr bool TE = BLK & 1, TM = BLK & 2;
    static constexpr int NC = ncomp<BLK>();
    static constexpr int ZC = BLK == 2 ? 0 : 2;   // local slot of Ez
    static constexpr int RX = 64 * CPL, RY = NW * R, NTH = 64 * NW;
    static constexpr int UP = up_rows<BLK>(), DN = dn_rows<BLK>();
    using V = Cols<T, CPL>;

    // LDS: [buffer][wavefront][UP + DN rows][64 lanes] of V
    static __device__ __forceinline__ V *row(void *lds, int buf, int w, int q)
    {
        return reinterpret_cast<V *>(lds) + ((size_t)(buf * NW + w) * (UP + DN) + q) * 64;
    }
    static __device__ __forceinline__ void put(V *p, int lane, const T (&v)[CPL])
    {
        V s;
#pragma unroll
        for (int c = 0; c < CPL; c++) s.v[c] = v[c];
        p[lane] = s;
    }
    static __device__ __forceinline__ void get(const V *p, int lane, T (&v)[CPL])
    {
        const V s = p[lane];
#pragma unroll
        for (int c = 0; c < CPL; c++) v[c] = s.v[c];
    }
    static __device__ __forceinline__ void put_up(void *lds, int buf, int w, int lane, const T (&x)[NC][R][CPL])
    {
        if (TE) put(row(lds, buf, w, 0), lane, x[0][0]);
        if (TM) put(row(lds, buf, w, UP - 1), lane, x[ZC][0]);
    }
    static __device__ __forceinline__ void put_dn(void *lds, int buf, int w, int lane, const T (&x)[NC][R][CPL])
    {
#pragma unroll
        for (int q = 0; q < DN; q++) put(row(lds, buf, w, UP + q), lane, x[q][R - 1]);
    }

    static __device__ __forceinline__ void derive(const T (&x)[NC][R][CPL], int j, Row<T, CPL> &r)
    {
#pragma unroll
        for (int c = 0; c < CPL; c++) {
            if (TE) {
                const T ey = x[1][j][c], eyp = right_of<T, CPL>(x[1][j], c);
                r.ex[c] = x[0][j][c];
                r.wg[c] = eyp - ey;
                r.h[c] = x[0][j][c] - left_of<T, CPL>(x[0][j], c);
                r.ly[c] = d2(left_of<T, CPL>(x[1][j], c), ey, eyp);
            }
            if (TM) {
                r.ez[c] = x[ZC][j][c];
                r.lx[c] = d2(left_of<T, CPL>(x[ZC][j], c), x[ZC][j][c], right_of<T, CPL>(x[ZC][j], c));
            }
        }
    }

    // One sweep in place: x <- b + A x on every row the wavefront holds,
    // neighbour rows from LDS buffer `rd`, the new first and last rows
    // published in buffer rd ^ 1 (the caller's barrier follows).
    static __device__ __forceinline__ void sweep(const Coef<T> &k, T (&x)[NC][R][CPL], const T (&b)[NC][R][CPL], void *lds,
                                                 int rd, int w, int lane)
    {
        const int wm = w > 0 ? w - 1 : 0, wp = w + 1 < NW ? w + 1 : NW - 1;
        Row<T, CPL> pm, cur, nx;
        {
            // previous row: the last row of the wavefront before
            T e[3][CPL];
#pragma unroll
            for (int q = 0; q < DN; q++) get(row(lds, rd, wm, UP + q), lane, e[q]);
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                if (TE) {
                    pm.ex[c] = e[0][c];
                    pm.wg[c] = right_of<T, CPL>(e[1], c) - e[1][c];
                }
                if (TM) {
                    pm.ez[c] = e[ZC][c];
                    pm.lx[c] = d2(left_of<T, CPL>(e[ZC], c), e[ZC][c], right_of<T, CPL>(e[ZC], c));
                }
            }
        }
        T ux[CPL], uz[CPL];
        if (TE) get(row(lds, rd, wp, 0), lane, ux);
        if (TM) get(row(lds, rd, wp, UP - 1), lane, uz);
        derive(x, 0, cur);
#pragma unroll
        for (int j = 0; j < R; j++) {
            if (j + 1 < R) {
                derive(x, j + 1, nx);
            } else {
#pragma unroll
                for (int c = 0; c < CPL; c++) {
                    if (TE) {
                        nx.ex[c] = ux[c];
                        nx.h[c] = ux[c] - left_of<T, CPL>(ux, c);
                    }
                    if (TM) {
                        nx.ez[c] = uz[c];
                        nx.lx[c] = d2(left_of<T, CPL>(uz, c), uz[c], right_of<T, CPL>(uz, c));
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                if (TE) {
                    const T vx = a_te_x_b(k.cxx, k.cxy, d2(pm.ex[c], cur.ex[c], nx.ex[c]), cur.wg[c] - pm.wg[c], b[0][j][c]);
                    const T vy = a_te_y_b(k.cyy, k.cxy, cur.ly[c], nx.h[c] - cur.h[c], b[1][j][c]);
                    x[0][j][c] = vx;
                    x[1][j][c] = vy;
                }
                if (TM) {
                    const T vz = a_tm_b(k.czx, k.czy, k.czz, cur.lx[c], d2(pm.ez[c], cur.ez[c], nx.ez[c]),
                                        d2(pm.lx[c], cur.lx[c], nx.lx[c]), b[ZC][j][c]);
                    x[ZC][j][c] = vz;
                }
            }
            if (j == 0) put_up(lds, rd ^ 1, w, lane, x);
            pm = cur;
            cur = nx;
        }
        put_dn(lds, rd ^ 1, w, lane, x);
    }
};

// One pass.  RK_FRONT forms dE' from E, B and the filtered current, and
// stores B^{n+1/2}, dE' and the iterate; RK_MID reads dE' and the iterate
// and stores the iterate; RK_LAST adds its iterate to E and, where asked to,
// hands the own cells of B back to the caller's buffers.  The front reads E
// of neighbouring tiles, so a step takes at least two passes.
template <typename T, int BLK, int CPL, int R, int NW, int KIND>
__global__ __launch_bounds__(64 * NW) void k2_reg(Coef<T> c, RegArgs<T> a, int ntx, int W, int H, int nwg)
{
    using G = Tile<T, BLK, CPL, R, NW>;
    constexpr bool FRONT = KIND == RK_FRONT, LAST = KIND == RK_LAST;
    constexpr bool TE = G::TE, TM = G::TM;
    constexpr int NC = G::NC, ZC = G::ZC;
    __shared__ __attribute__((aligned(16))) char lds[lds_bytes<T, BLK, CPL, NW>()];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wid = xcd_map(blockIdx.x, nwg);
    const int tx = wid % ntx, ty = wid / ntx;
    const int nx = c.nx, ny = c.ny;
    // first column and row of the region; output cells [X0, X0 + W) x [Y0, Y0 + H)
    const int X0 = tx * W, Y0 = ty * H;
    const int hx = a.k + (FRONT ? 1 : 0);
    const int gx0 = X0 - hx + lane * CPL, gy0 = Y0 - a.k + w * R;
    const unsigned rowb = (unsigned)nx * (unsigned)sizeof(T);
    unsigned colb[CPL];
    bool outc[CPL];
#pragma unroll
    for (int q = 0; q < CPL; q++) {
        const int g = gx0 + q;
        colb[q] = (unsigned)front2d::wrapi(g, nx) * (unsigned)sizeof(T);
        outc[q] = g >= X0 && g < X0 + W && g < nx;
    }
    const int yend = min(Y0 + H, ny);
    T x[NC][R][CPL], b[NC][R][CPL];
    if constexpr (FRONT) {
        const T sixth = c.lumped ? T(0) : T(1.0 / 6.0);
        // Rows -1 .. R + 1 of E and -1 .. R of B around the wavefront's rows;
        // B^{n+1/2} of rows -1 and R is recomputed by each wavefront instead
        // of exchanged
        T e1[3][CPL], bo1[3][CPL];
        T bz[2][CPL], by[3][CPL], byl[3][CPL], axbx[2][CPL], dxbz[CPL];
        int gy = front2d::wrapi(gy0 - 1, ny);
#pragma unroll
        for (int r = -1; r <= R + 1; r++) {
            const unsigned ro = (unsigned)gy * rowb;
            T e0[3][CPL], bo0[3][CPL];
#pragma unroll
            for (int q = 0; q < CPL; q++) {
                const unsigned o = ro + colb[q];
                if (TE) {
                    e0[0][q] = ld_off(a.E[0], o);
                    if (r <= R) e0[1][q] = ld_off(a.E[1], o);
                    if (r <= R) bo0[2][q] = ld_off(a.Bin[2], o);
                }
                if (TM) {
                    e0[2][q] = ld_off(a.E[2], o);
                    if (r <= R) {
                        bo0[0][q] = ld_off(a.Bin[0], o);
                        bo0[1][q] = ld_off(a.Bin[1], o);
                    }
                }
            }
            gy = gy + 1 < ny ? gy + 1 : 0;
            if (r >= 0) {
                // B^{n+1/2} of row r - 1
                const int s = r - 1;
                T bp[3][CPL];
#pragma unroll
                for (int q = 0; q < CPL; q++) {
                    if (TM) {
                        bp[0][q] = bo1[0][q] - c.tdy * (e0[2][q] - e1[2][q]);
                        bp[1][q] = bo1[1][q] + c.tdx * (right_of<T, CPL>(e1[2], q) - e1[2][q]);
                    }
                    if (TE)
                        bp[2][q] = bo1[2][q] - (c.tdx * (right_of<T, CPL>(e1[1], q) - e1[1][q]) -
                                                c.tdy * (e0[0][q] - e1[0][q]));
                }
                if (s >= 0 && s < R) {
                    const int g = gy0 + s;
                    if (g >= Y0 && g < yend)
#pragma unroll
                        for (int q = 0; q < CPL; q++)
                            if (outc[q]) {
                                const unsigned o = (unsigned)g * rowb + (unsigned)(gx0 + q) * (unsigned)sizeof(T);
                                if (TM) { st_off(a.B[0], o, bp[0][q]); st_off(a.B[1], o, bp[1][q]); }
                                if (TE) st_off(a.B[2], o, bp[2][q]);
                            }
                }
                T axn[CPL], dxn[CPL];
#pragma unroll
                for (int q = 0; q < CPL; q++) {
                    if (TM) {
                        axn[q] = avg6(left_of<T, CPL>(bp[0], q), bp[0][q], right_of<T, CPL>(bp[0], q), sixth);
                        by[0][q] = by[1][q]; by[1][q] = by[2][q]; by[2][q] = bp[1][q];
                        byl[0][q] = byl[1][q]; byl[1][q] = byl[2][q]; byl[2][q] = left_of<T, CPL>(bp[1], q);
                    }
                    if (TE) dxn[q] = bp[2][q] - left_of<T, CPL>(bp[2], q);
                }
                if (r >= 2) {
                    // dE' of row r - 2 (B^{n+1/2} rows r - 3 .. r - 1)
                    const int j = r - 2;
#pragma unroll
                    for (int q = 0; q < CPL; q++) {
                        T jf[3] = {T(0), T(0), T(0)};
                        if (a.Jf[0] != nullptr) {
                            int gj = gy0 + j;
                            gj = front2d::wrapi(gj, ny);
                            const unsigned o = (unsigned)gj * rowb + colb[q];
                            if (TE) { jf[0] = ld_off(a.Jf[0], o); jf[1] = ld_off(a.Jf[1], o); }
                            if (TM) jf[2] = ld_off(a.Jf[2], o);
                        }
                        if (TE) {
                            b[0][j][q] = c.tdy * (bz[1][q] - bz[0][q]) - a.env_src * jf[0];
                            b[1][j][q] = -c.tdx * dxbz[q] - a.env_src * jf[1];
                        }
                        if (TM) {
                            const T ay = avg6(by[0][q], by[1][q], by[2][q], sixth);
                            const T ayl = avg6(byl[0][q], byl[1][q], byl[2][q], sixth);
                            b[ZC][j][q] = c.tdx * (ay - ayl) - c.tdy * (axbx[1][q] - axbx[0][q]) - a.env_src * jf[2];
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < CPL; q++) {
                    if (TM) { axbx[0][q] = axbx[1][q]; axbx[1][q] = axn[q]; }
                    if (TE) { bz[0][q] = bz[1][q]; bz[1][q] = bp[2][q]; dxbz[q] = dxn[q]; }
                }
            }
#pragma unroll
            for (int q = 0; q < CPL; q++)
#pragma unroll
                for (int u = 0; u < 3; u++) { e1[u][q] = e0[u][q]; bo1[u][q] = bo0[u][q]; }
        }
#pragma unroll
        for (int u = 0; u < NC; u++)
#pragma unroll
            for (int j = 0; j < R; j++)
#pragma unroll
                for (int q = 0; q < CPL; q++) x[u][j][q] = b[u][j][q];
#pragma unroll
        for (int j = 0; j < R; j++) {
            const int g = gy0 + j;
            if (g < Y0 || g >= yend) continue;
#pragma unroll
            for (int q = 0; q < CPL; q++)
                if (outc[q]) {
                    const unsigned o = (unsigned)g * rowb + (unsigned)(gx0 + q) * (unsigned)sizeof(T);
                    if (TE) { st_off(a.dEp[0], o, b[0][j][q]); st_off(a.dEp[1], o, b[1][j][q]); }
                    if (TM) st_off(a.dEp[2], o, b[ZC][j][q]);
                }
        }
    } else {
        int gy = front2d::wrapi(gy0, ny);
#pragma unroll
        for (int j = 0; j < R; j++) {
            const unsigned ro = (unsigned)gy * rowb;
#pragma unroll
            for (int q = 0; q < CPL; q++) {
                const unsigned o = ro + colb[q];
#pragma unroll
                for (int u = 0; u < NC; u++) {
                    const int g = BLK == 2 ? 2 : u;
                    b[u][j][q] = ld_off(a.rhs[g], o);
                    x[u][j][q] = ld_off(a.x_in[g], o);
                }
            }
            gy = gy + 1 < ny ? gy + 1 : 0;
        }
    }
    G::put_up(lds, 0, w, lane, x);
    G::put_dn(lds, 0, w, lane, x);
    lds_barrier();
    for (int l = 0; l < a.k; l++) {
        G::sweep(c, x, b, lds, l & 1, w, lane);
        lds_barrier();
    }
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int g = gy0 + j;
        if (g < Y0 || g >= yend) continue;
#pragma unroll
        for (int q = 0; q < CPL; q++) {
            if (!outc[q]) continue;
            const unsigned o = (unsigned)g * rowb + (unsigned)(gx0 + q) * (unsigned)sizeof(T);
#pragma unroll
            for (int u = 0; u < NC; u++) {
                const int gc = BLK == 2 ? 2 : u;
                if (LAST) st_off(a.E[gc], o, ld_off(a.E[gc], o) + x[u][j][q]);
                else st_off(a.x_out[gc], o, x[u][j][q]);
            }
            if (LAST) {
                if (TE && a.Bd[2] != nullptr) st_off(a.Bd[2], o, ld_off(a.Bs[2], o));
                if (TM && a.Bd[0] != nullptr) {
                    st_off(a.Bd[0], o, ld_off(a.Bs[0], o));
                    st_off(a.Bd[1], o, ld_off(a.Bs[1], o));
                }
            }
        }
    }
}

template <typename T, int BLK, int CPL, int R, int NW, int KIND>
hipError_t launch_kind(const Coef<T> &c, const RegArgs<T> &a, hipStream_t s)
{
    using G = Tile<T, BLK, CPL, R, NW>;
    const int W = G::RX - 2 * a.k - (KIND == RK_FRONT ? 3 : 0), H = G::RY - 2 * a.k;
    if (W < 1 || H < 1) return hipErrorInvalidValue;
    const int ntx = (c.nx + W - 1) / W, n = ntx * ((c.ny + H - 1) / H);
    hipLaunchKernelGGL((k2_reg<T, BLK, CPL, R, NW, KIND>), dim3(n), dim3(G::NTH), 0, s, c, a, ntx, W, H, n);
    return hipGetLastError();
}

template <typename T, int BLK, int CPL, int R, int NW>
hipError_t launch_geo(const Coef<T> &c, int kind, const RegArgs<T> &a, hipStream_t s)
{
    switch (kind) {
    case RK_FRONT: return launch_kind<T, BLK, CPL, R, NW, RK_FRONT>(c, a, s);
    case RK_MID: return launch_kind<T, BLK, CPL, R, NW, RK_MID>(c, a, s);
    case RK_LAST: return launch_kind<T, BLK, CPL, R, NW, RK_LAST>(c, a, s);
    default: return hipErrorInvalidValue;
    }
}

// one pass of block set BLK on the geometry `geo` (index into the list of
// reg_geometry)
template <typename T, int BLK>
hipError_t launch(const Coef<T> &c, int geo, int kind, const RegArgs<T> &a, hipStream_t s)
{
    switch (geo) {
    case 0: return launch_geo<T, BLK, 1, 2, 16>(c, kind, a, s);
    case 1: return launch_geo<T, BLK, 1, 4, 8>(c, kind, a, s);
    case 2: return launch_geo<T, BLK, 1, 4, 16>(c, kind, a, s);
    case 3:
        if constexpr (BLK != 3) return launch_geo<T, BLK, 2, 4, 16>(c, kind, a, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

}  // namespace reg2d
}  // namespace mx
