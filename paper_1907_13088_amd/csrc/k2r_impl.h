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
// The TE and TM blocks share nothing but their launches: a launch over both
// deals each workgroup one block, so the blocks fill the CUs together and a
// tolerance solve stops them apart.  (Both blocks in each
// workgroup measured no faster: 1024^2 FP32, 20 sweeps, 57 against 56 us,
// 2048^2 165 against 159, 128^2 19 against 13.)
//
// Every value is formed by the operations of the row-streaming and LDS-tile
// kernels in the same order, so all schedules give bitwise equal fields.
//
// Bound: VALU issue (FP32, four rows per lane: 15 VALU instructions per TE
// cell and sweep and 13 per TM cell, with 1 and 0.75 LDS accesses; 1500 x 1100,
// 64 x 64 regions: 2.4 us per sweep of both blocks, near the issue limit of 6
// million region cells), and below that the latency of a sweep (0.2 to 0.5
// us) and the 3 to 6 us of a launch with its loads and stores.  What it
// replaced was bound by latency: the LDS-tile kernel ran 128^2 on 32
// workgroups, a row stream of 1024^2 has one wavefront per SIMD and pays
// about 1 us per row.
#include <algorithm>

#include "k2f_impl.h"
#include "mx_internal.h"
#include "stencil2d.h"

namespace mx {
namespace reg2d {

using front2d::avg6;

// value of column c - 1 / c + 1 of a lane's row of CPL columns
template <typename T, int CPL>
__device__ __forceinline__ T left_of(const T (&v)[CPL], int c) { return c > 0 ? v[c > 0 ? c - 1 : 0] : from_left(v[CPL - 1]); }
template <typename T, int CPL>
__device__ __forceinline__ T right_of(const T (&v)[CPL], int c)
{
    return c + 1 < CPL ? v[c + 1 < CPL ? c + 1 : 0] : from_right(v[0]);
}

template <int BLK> constexpr int ncomp() { return BLK == 1 ? 2 : 1; }   // 1 TE, 2 TM

// CPL values of one lane, one LDS access
template <typename T, int CPL>
struct alignas(CPL * sizeof(T)) Cols {
    T v[CPL];
};

// LDS rows a wavefront publishes per sweep: its first row (Ex, or Ez: the next
// row of the wavefront before it) and its last row (Ex and Ey, or Ez: the
// previous row of the wavefront after it)
template <typename T, int CPL, int NW>
constexpr size_t lds_bytes() { return sizeof(T) * 2 * NW * 3 * 64 * CPL; }   // TE's, the larger

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
    static constexpr int YC = TE ? 1 : 0, ZC = 0;   // local slots of Ey and Ez
    static constexpr int RX = 64 * CPL, RY = NW * R, NTH = 64 * NW;
    static constexpr int UP = 1, DN = NC;
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

    // One sweep in place on every row the wavefront holds, neighbour rows from
    // LDS buffer `rd`, the new first and last rows published in buffer rd ^ 1
    // (the caller's barrier follows).  Standard form: x <- b + A x.  Delta
    // form: x <- A x, b <- b + x (b the running sum).  Chebyshev form: r = b +
    // A x - x, d <- f d + g r, x <- x + d.  RES: the squares of the step (the
    // residual in the Chebyshev form) of the cells `in` (bit j CPL + c) are
    // added to nrm.
    template <int FORM, bool RES>
    static __device__ __forceinline__ void sweep(const Coef<T> &k, T (&x)[NC][R][CPL], T (&b)[NC][R][CPL], T (&d)[NC][R][CPL],
                                                 T cf, T cg, void *lds, int rd, int w, int lane, unsigned in, double &nrm)
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
                constexpr bool PLAIN = FORM == FM_DELTA;
                T v[NC];
                if (TE) {
                    const T lyy = d2(pm.ex[c], cur.ex[c], nx.ex[c]), dg = cur.wg[c] - pm.wg[c], dh = nx.h[c] - cur.h[c];
                    v[0] = PLAIN ? a_te_x(k.cxx, k.cxy, lyy, dg) : a_te_x_b(k.cxx, k.cxy, lyy, dg, b[0][j][c]);
                    v[YC] = PLAIN ? a_te_y(k.cyy, k.cxy, cur.ly[c], dh) : a_te_y_b(k.cyy, k.cxy, cur.ly[c], dh, b[YC][j][c]);
                }
                if (TM) {
                    const T ly = d2(pm.ez[c], cur.ez[c], nx.ez[c]), lxy = d2(pm.lx[c], cur.lx[c], nx.lx[c]);
                    v[ZC] = PLAIN ? a_tm(k.czx, k.czy, k.czz, cur.lx[c], ly, lxy) : a_tm_b(k.czx, k.czy, k.czz, cur.lx[c], ly, lxy, b[ZC][j][c]);
                }
#pragma unroll
                for (int u = 0; u < NC; u++) {
                    const T xo = x[u][j][c];
                    T r = v[u];
                    if (FORM == FM_DELTA) b[u][j][c] += v[u];
                    if (FORM == FM_CHEB) {
                        r = v[u] - xo;
                        d[u][j][c] = fmad(cf, d[u][j][c], cg * r);
                        v[u] = xo + d[u][j][c];
                    }
                    if (RES && (in >> (j * CPL + c) & 1)) {
                        const double e = FORM == FM_STD ? (double)v[u] - (double)xo : (double)r;
                        nrm += e * e;
                    }
                    x[u][j][c] = v[u];
                }
            }
            if (j == 0) put_up(lds, rd ^ 1, w, lane, x);
            pm = cur;
            cur = nx;
        }
        put_dn(lds, rd ^ 1, w, lane, x);
    }
};

// Sum of a double over a wavefront in a fixed order (valid in every lane): row
// scans and row broadcasts by DPP, a fifth of the latency of lane shuffles
__device__ __forceinline__ double wave_sum(double v)
{
    v += lane_dpp<0x111>(v);          // row_shr:1
    v += lane_dpp<0x112>(v);          // row_shr:2
    v += lane_dpp<0x114>(v);          // row_shr:4
    v += lane_dpp<0x118>(v);          // row_shr:8: the last lane of a row holds the row's sum
    v += lane_dpp<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
    v += lane_dpp<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3: the last lane holds all
    const long long u = __builtin_bit_cast(long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((int)u, 63), hi = __builtin_amdgcn_readlane((int)(u >> 32), 63);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Tolerance solve: the norms the launch before left per workgroup are summed
// by one wavefront of every workgroup of this launch in the same order, so
// all of them take the same stop decision and no launch is spent on it (the
// workgroup's other wavefronts load their tile meanwhile); the block's first
// workgroup keeps the state for the launches that follow.
__device__ __forceinline__ RegTolBlock reg_tol_decide(const RegTol &t, int b)
{
    RegTolBlock s = t.state[(t.par ^ 1) * 2 + b];
    if (t.init) s = RegTolBlock{0.0, 0.0, 0, 0, 0, -1, 0, 0};
    if ((t.init || t.test) && !s.skip) {
        const double *p0 = t.norms + (size_t)b * t.stride, *p1 = t.norms + (size_t)(2 + 2 * (t.par ^ 1) + b) * t.stride;
        double n0 = 0.0, n1 = 0.0;
        // four workgroups' values a lane at a time, their loads in flight
        // together (of the list not asked for too: it is not used)
        for (int i0 = threadIdx.x & 63; i0 < t.npart; i0 += 256) {
            double v0[4], v1[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int i = min(i0 + 64 * u, t.npart - 1);
                v0[u] = p0[i];
                v1[u] = p1[i];
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (i0 + 64 * u < t.npart) {
                    n0 += v0[u];
                    n1 += v1[u];
                }
        }
        if (t.init) {
            s.rhsn = sqrt(wave_sum(n0));
            if (!isfinite(s.rhsn)) s.nonfinite = 1;
            if (!(s.rhsn > 0.0) || s.nonfinite) s.skip = 1;   // dE' = 0: the increment is 0, no sweeps
        }
        if (t.test && !s.skip) {
            s.resid = sqrt(wave_sum(n1));
            s.done += t.kk;
            s.last = t.buf;
            if (!isfinite(s.resid)) {
                s.nonfinite = 2;
                s.skip = 1;
            } else if (s.resid <= t.tol * s.rhsn) {
                s.conv = 1;
                s.skip = 1;
            }
        }
    }
    return s;
}

// One pass of block BLK on the tile of workgroup `wid` (of the block's).
// RK_FRONT forms dE' from E, B and the filtered current, and stores
// B^{n+1/2}, dE' and the iterate; RK_MID reads dE' and the iterate and stores
// the iterate; RK_LAST adds its iterate to E and, where asked to, hands the
// own cells of B back to the caller's buffers.  The front reads E of
// neighbouring tiles, so a step takes at least two passes.  TOL: the pass
// also leaves the squared norms of dE' (front) and, if asked to, of its last
// sweep's step.
template <typename T, int BLK, int CPL, int R, int NW, int KIND, int FORM, bool TOL>
__device__ __forceinline__ void reg_pass(const Coef<T> &c, const RegArgs<T> &a, int ntx, int W, int H, int wid, void *lds, double (*sh)[2],
                                         int *stop)
{
    using G = Tile<T, BLK, CPL, R, NW>;
    constexpr bool FRONT = KIND == RK_FRONT, LAST = KIND == RK_LAST;
    constexpr bool TE = G::TE, TM = G::TM;
    constexpr int NC = G::NC, YC = G::YC, ZC = G::ZC;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
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
    const bool first = FRONT || a.first;
    const bool halt = TOL && *a.tol.stall == a.tol.epoch;
    T x[NC][R][CPL], b[NC][R][CPL], d[NC][R][CPL];
    double nb = 0.0, nr = 0.0;   // squared norms of dE' and of the last step
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
                // (an earlier step of the queue waits for the host: nothing is
                // stored)
                if (TOL && s == -1 && halt) return;
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
                            b[YC][j][q] = -c.tdx * dxbz[q] - a.env_src * jf[1];
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
                for (int q = 0; q < CPL; q++) {
                    x[u][j][q] = b[u][j][q];
                    d[u][j][q] = T(0);
                }
#pragma unroll
        for (int j = 0; j < R; j++) {
            const int g = gy0 + j;
            if (g < Y0 || g >= yend) continue;
#pragma unroll
            for (int q = 0; q < CPL; q++)
                if (outc[q]) {
                    const unsigned o = (unsigned)g * rowb + (unsigned)(gx0 + q) * (unsigned)sizeof(T);
                    if (TE) { st_off(a.dEp[0], o, b[0][j][q]); st_off(a.dEp[1], o, b[YC][j][q]); }
                    if (TM) st_off(a.dEp[2], o, b[ZC][j][q]);
                    if (TOL)
#pragma unroll
                        for (int u = 0; u < NC; u++) nb += (double)b[u][j][q] * (double)b[u][j][q];
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
                    x[u][j][q] = ld_off(a.x_in[g], o);
                    // the running sum of cells that neighbouring tiles own may
                    // already be theirs of this pass: it is not used
                    b[u][j][q] = ld_off(FORM == FM_DELTA && !first ? a.s_in[g] : a.rhs[g], o);
                    if (FORM == FM_CHEB) d[u][j][q] = first ? T(0) : ld_off(a.s_in[g], o);
                }
            }
            gy = gy + 1 < ny ? gy + 1 : 0;
        }
    }
    constexpr int bk = BLK - 1;
    if constexpr (TOL && !FRONT) {
        if (w == 0) {
            const RegTolBlock s = reg_tol_decide(a.tol, bk);
            if (lane == 0) {
                *stop = s.skip || halt;
                if (wid == 0 && !halt) a.tol.state[a.tol.par * 2 + bk] = s;
            }
        }
    }
    G::put_up(lds, 0, w, lane, x);
    G::put_dn(lds, 0, w, lane, x);
    lds_barrier();
    if constexpr (TOL && !FRONT)
        if (*stop) return;   // the block has met its stop test, or the queue halts
    const int kplain = TOL && a.tol.res ? a.k - 1 : a.k;
    for (int l = 0; l < kplain; l++) {
        G::template sweep<FORM, false>(c, x, b, d, a.cheb[bk][0][l], a.cheb[bk][1][l], lds, l & 1, w, lane, 0u, nr);
        lds_barrier();
    }
    if constexpr (TOL) {
        static_assert(R * CPL <= 32, "a bit per cell");
        if (a.tol.res) {
            unsigned in = 0;
#pragma unroll
            for (int j = 0; j < R; j++)
#pragma unroll
                for (int q = 0; q < CPL; q++)
                    if (outc[q] && gy0 + j >= Y0 && gy0 + j < yend) in |= 1u << (j * CPL + q);
            G::template sweep<FORM, true>(c, x, b, d, a.cheb[bk][0][kplain], a.cheb[bk][1][kplain], lds, kplain & 1, w, lane, in, nr);
        }
        // ahead of the tile's stores: nothing here waits for memory
        if (FRONT) nb = wave_sum(nb);
        nr = wave_sum(nr);
        if (lane == 0) {
            sh[w][0] = nb;
            sh[w][1] = nr;
        }
        lds_barrier();
        if (threadIdx.x == 0) {
            double s0 = 0.0, s1 = 0.0;
            for (int i = 0; i < NW; i++) {
                s0 += sh[i][0];
                s1 += sh[i][1];
            }
            if (FRONT) a.tol.norms[(size_t)bk * a.tol.stride + wid] = s0;
            a.tol.norms[(size_t)(2 + 2 * a.tol.par + bk) * a.tol.stride + wid] = s1;
        }
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
                else {
                    st_off(a.x_out[gc], o, x[u][j][q]);
                    if (FORM == FM_DELTA) st_off(a.s_out[gc], o, b[u][j][q]);
                    if (FORM == FM_CHEB) st_off(a.s_out[gc], o, d[u][j][q]);
                }
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

// Launch over the blocks of `mask` (1 TE, 2 TM, 3 both: the first n
// workgroups TE, the rest TM)
// At most 80 scalar and, where the cells leave room, 64 vector registers:
// above, a SIMD holds seven wavefronts instead of eight and a CU one workgroup
// of 1024 threads instead of two (1500 x 1100 FP32, 64 x 64 regions, 8 sweeps,
// by the scalar ones: front 52 -> 38 us, tested pass 43 -> 33).
template <typename T, int CPL, int R, int FORM>
constexpr int min_waves() { return R * CPL * 2 * (FORM == FM_CHEB ? 3 : 2) * (int)sizeof(T) / 4 <= 32 ? 8 : 4; }
template <typename T, int CPL, int R, int NW, int KIND, int FORM, bool TOL>
__global__ __launch_bounds__(64 * NW, (min_waves<T, CPL, R, FORM>())) __attribute__((amdgpu_num_sgpr(80))) void k2_reg(Coef<T> c, RegArgs<T> a, int mask, int ntx, int W, int H, int n)
{
    __shared__ __attribute__((aligned(16))) char lds[lds_bytes<T, CPL, NW>()];
    __shared__ double sh[TOL ? NW : 1][2];
    __shared__ int stop;
    const int id = xcd_map(blockIdx.x, gridDim.x);
    const bool tm = mask == 2 || id >= n;
    const int wid = id >= n ? id - n : id;
    if (tm) reg_pass<T, 2, CPL, R, NW, KIND, FORM, TOL>(c, a, ntx, W, H, wid, lds, sh, &stop);
    else reg_pass<T, 1, CPL, R, NW, KIND, FORM, TOL>(c, a, ntx, W, H, wid, lds, sh, &stop);
}

template <typename T, int CPL, int R, int NW, int KIND, int FORM, bool TOL>
hipError_t launch_kind(const Coef<T> &c, int mask, const RegArgs<T> &a, hipStream_t s, int *npart)
{
    constexpr int RX = 64 * CPL, RY = NW * R;
    const int W = RX - 2 * a.k - (KIND == RK_FRONT ? 3 : 0), H = RY - 2 * a.k;
    if (W < 1 || H < 1 || a.k > 16) return hipErrorInvalidValue;
    const int ntx = (c.nx + W - 1) / W, n = ntx * ((c.ny + H - 1) / H);
    if (TOL && n > a.tol.stride) return hipErrorInvalidValue;
    if (npart) *npart = n;
    hipLaunchKernelGGL((k2_reg<T, CPL, R, NW, KIND, FORM, TOL>), dim3(mask == 3 ? 2 * n : n), dim3(64 * NW), 0, s, c, a,
                       mask, ntx, W, H, n);
    return hipGetLastError();
}

template <typename T, int CPL, int R, int NW, int FORM, bool TOL>
hipError_t launch_geo(const Coef<T> &c, int mask, int kind, const RegArgs<T> &a, hipStream_t s, int *npart)
{
    if (kind == RK_FRONT) return launch_kind<T, CPL, R, NW, RK_FRONT, FORM, TOL>(c, mask, a, s, npart);
    if (kind == RK_MID) return launch_kind<T, CPL, R, NW, RK_MID, FORM, TOL>(c, mask, a, s, npart);
    if constexpr (!TOL)
        if (kind == RK_LAST) return launch_kind<T, CPL, R, NW, RK_LAST, FORM, TOL>(c, mask, a, s, npart);
    return hipErrorInvalidValue;
}

// one pass over the blocks of `mask` on the geometry `geo` (index into GEO of
// plan2r.h); *npart receives the workgroups per block
template <typename T, int FORM, bool TOL>
hipError_t launch(const Coef<T> &c, int mask, int geo, int kind, const RegArgs<T> &a, hipStream_t s, int *npart)
{
    if (mask < 1 || mask > 3) return hipErrorInvalidValue;
    switch (geo) {
    case 0: return launch_geo<T, 1, 2, 16, FORM, TOL>(c, mask, kind, a, s, npart);
    case 1: return launch_geo<T, 1, 4, 8, FORM, TOL>(c, mask, kind, a, s, npart);
    case 2: return launch_geo<T, 1, 4, 16, FORM, TOL>(c, mask, kind, a, s, npart);
    case 3:
        if constexpr (sizeof(T) == 4) return launch_geo<T, 2, 4, 16, FORM, TOL>(c, mask, kind, a, s, npart);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

}  // namespace reg2d
}  // namespace mx
