// 3D mass-matrix sweep pass, K sweeps per pass over HBM (Alg 1 with A from
// eqs matrixA_1st..matrixA_last; the Chebyshev form of the accelerated
// solve), marching in z.
//
// The 33-point A of each component splits into quantities of one z plane
// (differences and averages across x and y) combined along z: e.g. the x
// component is
//   (A x)_x = a_yy Dyy X + a_zz Dzz X + a_yz Dzz(Dyy X) + o_xy avg_z(Dx Dy Y)
//           + o_xz (avg_y(Dx Z)(k) - avg_y(Dx Z)(k - 1)),
// so a sweep level needs only one plane of its input in LDS.  When plane p
// of a level's input arrives, its in-plane quantities are folded at once
// into the three outputs they touch (planes p - 1, p and p + 1): output
// p - 1 is then complete, and only two partial sums per column are carried
// instead of windows of the quantities themselves.  Every output is summed
// in the same order, ((from p - 1) + (from p)) + (from p + 1), whatever the
// pass depth, so passes of any depth give bitwise identical iterates.
//
// A workgroup of NW waves owns a column tile of 64 x TY (TY = R NW): lane =
// x column, wave w carries rows w R .. w R + R - 1 in registers.  Level l
// (1..K) computes plane t - 2l at march step t from the planes of level
// l - 1 that arrived at earlier steps (one barrier per step).  Neighbours
// across x come from the neighbouring lanes, rows above and below from the
// wave's own registers; LDS carries only the first and last row of each
// wave, in a buffer per level and parity.  The valid columns shrink by one
// per level on each side; along y the level-0 plane is loaded with one row
// more on each side.  So a tile writes (64 - 2K) x (TY - 2(K - 1)) columns, a
// wide one two more.
// The carried value (dE' in the standard form, the running sum in the delta
// form, dE' and the increment in the Chebyshev form) is read when level 1
// completes a plane and then travels with the planes.
//
// What bounds it: VALU issue and, with the 8 to 16 waves that fit a CU, the
// latencies between two barriers (512^3, FP32, three sweeps: 58 % of the VALU
// cycles; the HBM traffic alone would take half the time).  Rows in registers
// instead of planes in LDS take a quarter of the VALU and four fifths of the
// LDS instructions away against a kernel that reads the 3 x 3 columns of each
// point from LDS, which measured, per pass: 512^3 FP32 delta form 2.11 ms
// against 1.93 now, FP32 Alg 1 1.69 against 1.40 (ten sweeps, front taken
// off), 256^3 FP64 0.38 against 0.32, Chebyshev FP64 at 250^3 8.64 ms per
// step against 7.19.
// The first level has no neighbour for its outer lanes, which costs a tile two
// columns (58 instead of 60 in FP32 with three sweeps, 60 instead of 62 in FP64
// with two).  Where they add a column of tiles the wide tiles take those
// neighbours from memory: one load per plane and wave, spread to the two lanes
// by scalar reads, some 5 % of the pass (60 x 300 x 300 FP32, three sweeps, us per step:
// delta form 1871 narrow, 1274 wide, 1264 by the kernel that read every point from LDS;
// 62 x 300 x 300 FP64 6503, 4685, 4852; 180^3 FP32 delta 1424, 1326, 1331).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "mx_internal.h"
#include "plan3d.h"
#include "stencil2d.h"

namespace mx {
namespace {

__device__ __forceinline__ int wrapm(int i, int n)
{
    i %= n;
    return i < 0 ? i + n : i;
}

template <typename T>
struct P3 {
    T x, y, z;
};

template <typename T>
__device__ __forceinline__ P3<T> p3add(const P3<T> &a, const P3<T> &b)
{
    return P3<T>{a.x + b.x, a.y + b.y, a.z + b.z};
}

// z-independent factors of the three plane contributions, formed in FP64 on
// the host from the coefficients of A and rounded once
template <typename T>
struct Zc {
    // x, from planes p - 1 and p + 1: a01 X + a02 Dyy X + o2/6 DxDy Y
    //    (and - o1 rxz from p - 1); from p: (a00 - 2 a02) Dyy X - 2 a01 X
    //    + 2 o2/3 DxDy Y + o1 rxz
    T a01, a02, o2s, o1, b00, m01, o2c;
    // y: the same with the roles of x and y exchanged
    T a10, a12, o0, b11, m10;
    // z, from p: a20 Dxx Z + a21 Dyy Z + a22 DxxDyy Z - o1 szx - o0 szy;
    //    from p + 1: o1 szx + o0 szy
    T a20, a21, a22;
};

// in-plane quantities of one column of one plane (see the header comment)
template <typename T>
struct Q {
    T X, Y, Z;          // own values
    T lyyx, pxy, rxz;   // Dyy X, Dx Dy Y, avg_y(Dx Z)   (x component)
    T lxxy, pyx, ryz;   // Dxx Y, Dy Dx X, avg_x(Dy Z)   (y component)
    T lxxz, lyyz, lxyz; // Dxx Z, Dyy Z, Dyy Dxx Z       (z component)
    T szx, szy;         // avg_y(Dx' X), avg_x(Dy' Y)    (backward differences)
};

// average with weights (1, 4, 1)/6: f0 + (fm + fp - 2 f0)/6
template <typename T>
__device__ __forceinline__ T avg6(T fm, T f0, T fp)
{
    return fmad(d2(fm, f0, fp), T(1.0 / 6.0), f0);
}

// one row of a plane: its values and the differences along x that the rows
// above and below it use too
template <typename T>
struct Row {
    P3<T> v;
    T dx, dz, lxx;   // Dx' X (backward), Dx Z (forward), Dxx Z
};

// values of a row beyond the wave's first and last column
template <typename T>
struct Edge {
    P3<T> l, r;
};
// shifts with (W) and without such values
template <bool W, typename T>
__device__ __forceinline__ T left_of(T v, T edge)
{
    if constexpr (W) return from_left(v, edge);
    else return from_left(v);
}
template <bool W, typename T>
__device__ __forceinline__ T right_of(T v, T edge)
{
    if constexpr (W) return from_right(v, edge);
    else return from_right(v);
}

template <bool W, typename T>
__device__ __forceinline__ Row<T> row_of(const P3<T> &v, const Edge<T> &e)
{
    const T zr = right_of<W>(v.z, e.r.z);
    return Row<T>{v, v.x - left_of<W>(v.x, e.l.x), zr - v.z, d2(left_of<W>(v.z, e.l.z), v.z, zr)};
}

// the quantities of the middle one of three rows (em, ec, ep: their edges)
template <bool W, typename T>
__device__ __forceinline__ Q<T> inplane(const Row<T> &m, const Row<T> &c, const Row<T> &p, const Edge<T> &em, const Edge<T> &ec,
                                        const Edge<T> &ep)
{
    Q<T> q;
    q.X = c.v.x;
    q.Y = c.v.y;
    q.Z = c.v.z;
    const T dy = c.v.y - m.v.y, dyz = p.v.z - c.v.z, dyr = right_of<W>(dy, ec.r.y - em.r.y);
    q.lyyx = d2(m.v.x, c.v.x, p.v.x);
    q.pxy = dyr - dy;
    q.rxz = avg6(m.dz, c.dz, p.dz);
    q.lxxy = d2(left_of<W>(c.v.y, ec.l.y), c.v.y, right_of<W>(c.v.y, ec.r.y));
    q.pyx = p.dx - c.dx;
    q.ryz = avg6(left_of<W>(dyz, ep.l.z - ec.l.z), dyz, right_of<W>(dyz, ep.r.z - ec.r.z));
    q.lxxz = c.lxx;
    q.lyyz = d2(m.v.z, c.v.z, p.v.z);
    q.lxyz = d2(m.lxx, c.lxx, p.lxx);
    q.szx = avg6(m.dx, c.dx, p.dx);
    q.szy = avg6(left_of<W>(dy, ec.l.y - em.l.y), dy, dyr);
    return q;
}

// contributions of plane p to the outputs at p + 1 (f0), p (f1), p - 1 (f2)
template <typename T>
__device__ __forceinline__ void fold(const Zc<T> &z, const Q<T> &q, P3<T> &f0, P3<T> &f1, P3<T> &f2)
{
    const T sx = fmad(z.o2s, q.pxy, fmad(z.a02, q.lyyx, z.a01 * q.X));
    const T sy = fmad(z.o2s, q.pyx, fmad(z.a12, q.lxxy, z.a10 * q.Y));
    f2 = P3<T>{sx, sy, fmad(z.o1, q.szx, z.o0 * q.szy)};
    f0 = P3<T>{fmad(-z.o1, q.rxz, sx), fmad(-z.o0, q.ryz, sy), T(0)};
    f1.x = fmad(z.o1, q.rxz, fmad(z.o2c, q.pxy, fmad(z.m01, q.X, z.b00 * q.lyyx)));
    f1.y = fmad(z.o0, q.ryz, fmad(z.o2c, q.pyx, fmad(z.m10, q.Y, z.b11 * q.lxxy)));
    f1.z = fmad(-z.o0, q.szy, fmad(-z.o1, q.szx, fmad(z.a22, q.lxyz, fmad(z.a21, q.lyyz, z.a20 * q.lxxz))));
}

template <typename T>
__device__ __forceinline__ T comp(const P3<T> &p, int q) { return q == 0 ? p.x : (q == 1 ? p.y : p.z); }
template <typename T>
__device__ __forceinline__ void setc(P3<T> &p, int q, T v)
{
    if (q == 0) p.x = v;
    else if (q == 1) p.y = v;
    else p.z = v;
}

// FORM: FM_STD (x_l = b + A x_(l-1)), FM_DELTA (d_l = A d_(l-1), s_l = s_(l-1)
// + d_l) or FM_CHEB (r = b + A x - x, d_l = f_l d_(l-1) + g_l r, x_l = x + d_l).
// WIDE: the first level takes the columns beyond a wave's own from memory, so
// the valid columns shrink from the second level on.
template <typename T, int K, int FORM, bool LAST, int R, int NW, bool WIDE>
__global__ __launch_bounds__(64 * NW) void k3_stream(Coef<T> c, Zc<T> z, SweepArgs<T> a, int flags, int Lz)
{
    constexpr bool DELTA = FORM == FM_DELTA, CHEB = FORM == FM_CHEB;
    // rows at the waves' edges in LDS, EDGE per wave: wave w's first row in
    // slot EDGE w + 1, its last in slot EDGE w + EDGE; the first and the last
    // slot hold the rows around the tile (level 0 only)
    constexpr int TY = NW * R, EDGE = R > 1 ? 2 : 1, SLOTS = EDGE * NW + 2;
    static_assert(NW >= 2, "the first and the last wave load one row more each");
    if (a.skip && *a.skip) return;   // the solve has met its stop test
    __shared__ T pl[K][2][SLOTS][3][64];   // [level][parity][slot][component][x]
    __shared__ double sred[NW];
    const int nx = c.nx, ny = c.ny, nz = c.nz;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwg = gridDim.x * gridDim.y * gridDim.z;
    const int lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const int tl = xcd_map(lin, nwg);
    const int gxy = gridDim.x * gridDim.y;
    constexpr int HX = WIDE ? K - 1 : K;   // columns a pass loses on each side
    constexpr int OX = 64 - 2 * HX, OY = TY - 2 * (K - 1);   // output columns of a tile
    const int X0 = (tl % gridDim.x) * OX, Y0 = ((tl % gxy) / gridDim.x) * OY;
    const int Z0 = (tl / gxy) * Lz, Z1 = min(nz, Z0 + Lz);
    const size_t plane = (size_t)nx * ny;
    // own columns: x = ux, rows uy0 + r.  Plane and row are the same for a
    // wave, so each row of an array is a buffer with a scalar base, and the
    // lane's offset along x serves all of them.  An offset past the row's
    // end drops a store, without a branch: every step issues the same
    // memory operations, and the wait for a load leaves later stores alone.
    const int ux = X0 - HX + lane, uy0 = Y0 - (K - 1) + w * R;
    constexpr unsigned DROP = BUF_DROP;
    const unsigned row_bytes = (unsigned)nx * (unsigned)sizeof(T);
    const unsigned xin_off = (unsigned)wrapm(ux, nx) * (unsigned)sizeof(T);
    const unsigned xout_off = lane >= HX && lane < 64 - HX && ux < nx ? xin_off : DROP;
    size_t row[R];
    bool outy[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        row[r] = (size_t)wrapm(uy0 + r, ny) * nx;
        const int iy = w * R + r;
        outy[r] = iy >= K - 1 && iy < TY - (K - 1) && uy0 + r < ny;
    }
    const bool ring = w == 0 || w == NW - 1;   // waves that load a row around the tile
    const size_t rrow = (size_t)wrapm(w == 0 ? uy0 - 1 : uy0 + R, ny) * nx;
    const unsigned ring_off = ring ? xin_off : DROP;
    const int rslot = w == 0 ? 0 : SLOTS - 1;
    const bool first = flags & SW_FIRST, store = flags & SW_STORE, resid = flags & SW_RESID;
    const T *xin[3], *cin[3], *din[3];
#pragma unroll
    for (int q = 0; q < 3; q++) {
        xin[q] = first ? a.rhs[q] : a.x_in[q];
        cin[q] = (DELTA && !first) ? a.s_in[q] : a.rhs[q];
        din[q] = first ? a.rhs[q] : a.s_in[q];
    }
    const unsigned din_off = first ? DROP : xin_off;   // no increment yet: zero
    // WIDE: the edges of rows uy0 - 1 .. uy0 + R of a level-0 plane, one value
    // per lane (row, component, side), in one load
    const int er = min(lane / 6, R + 1), eq = (lane % 6) >> 1;
    const T *const ebase = (eq == 0 ? xin[0] : (eq == 1 ? xin[1] : xin[2])) + (size_t)wrapm(uy0 - 1 + er, ny) * nx +
                           wrapm(lane & 1 ? X0 - HX + 64 : X0 - HX - 1, nx);
    T en = T(0), ev = T(0);   // of the plane in flight, and of the newest one
    auto load3 = [&](const T *const (&f)[3], size_t o, unsigned at) {
        return P3<T>{buf_load(f[0] + o, row_bytes, at), buf_load(f[1] + o, row_bytes, at),
                     buf_load(f[2] + o, row_bytes, at)};
    };
    auto publish = [&](int l, int par, int slot, const P3<T> &v) {
        pl[l][par][slot][0][lane] = v.x;
        pl[l][par][slot][1][lane] = v.y;
        pl[l][par][slot][2][lane] = v.z;
    };
    // per level l (1..K) and row: partial sums of the outputs at planes p
    // (sa) and p + 1 (sb) after plane p of level l - 1 arrived, and the own
    // value (xp), carried value (cp) and increment (dp) of plane p, used when
    // output p completes; per level l (0..K-1): newest plane (val), and for
    // l >= 1 its carried value (oc) and increment (od), for level l + 1
    const P3<T> zero3{T(0), T(0), T(0)};
    P3<T> val[K][R], sa[K + 1][R], sb[K + 1][R], xp[K + 1][R], cp[K + 1][R], dp[K + 1][R], oc[K + 1][R], od[K + 1][R];
    P3<T> pe[R];   // E of the next output plane (last pass)
#pragma unroll
    for (int r = 0; r < R; r++) {
#pragma unroll
        for (int l = 0; l < K; l++) val[l][r] = zero3;
#pragma unroll
        for (int l = 0; l <= K; l++) sa[l][r] = sb[l][r] = xp[l][r] = cp[l][r] = dp[l][r] = oc[l][r] = od[l][r] = zero3;
        pe[r] = zero3;
    }
    double acc = 0.0;
    const int tbeg = Z0 - K, tend = Z1 + 2 * K, tout = Z0 + 2 * K;   // tout: level K completes plane Z0
    // level-0 plane in flight (own rows, row around the tile): loaded a step
    // before its use
    P3<T> px[R], pr;
    auto fetch = [&](int t, int zw) {
        const size_t zin = (size_t)zw * plane;
        const bool in = t < Z1 + K;
#pragma unroll
        for (int r = 0; r < R; r++) px[r] = load3(xin, zin + row[r], in ? xin_off : DROP);
        pr = load3(xin, zin + rrow, in ? ring_off : DROP);
        if (WIDE) en = ebase[zin];
    };
    int zt = wrapm(tbeg, nz), ze = wrapm(tbeg + 1 - 2 * K, nz);   // planes t and t + 1 - 2K, wrapped
    auto step = [&](const int t, auto out_) {
        constexpr bool OUT = decltype(out_)::value;   // level K completes a plane of the chunk
        const int pw = (t - tbeg) & 1, prd = pw ^ 1;
#pragma unroll
        for (int l = K; l >= 1; l--) {
            // arrival of plane p = t - 2l + 1 of level l - 1 (written at the
            // previous step); it completes output o = p - 1 of level l (before
            // the first that level l + 1 takes: a value that nothing reads)
            const int p = t - 2 * l + 1, o = p - 1;
            if ((OUT && l == K) || (p >= Z0 - (K - l + 1) && p < Z1 + (K - l + 1))) {
                auto edge = [&](int slot) {
                    return P3<T>{pl[l - 1][prd][slot][0][lane], pl[l - 1][prd][slot][1][lane],
                                 pl[l - 1][prd][slot][2][lane]};
                };
                const P3<T> below = edge(EDGE * w + EDGE + 1);
                const P3<T> above = edge(EDGE * w);
                // edges of the row in slot i (0: the row above the wave's first)
                auto side = [&](int i) {
                    Edge<T> e{};
                    if (WIDE && l == 1) {
                        e.l = P3<T>{lane_read(ev, 6 * i), lane_read(ev, 6 * i + 2), lane_read(ev, 6 * i + 4)};
                        e.r = P3<T>{lane_read(ev, 6 * i + 1), lane_read(ev, 6 * i + 3), lane_read(ev, 6 * i + 5)};
                    }
                    return e;
                };
                auto row_at = [&](const P3<T> &v, const Edge<T> &e) { return WIDE && l == 1 ? row_of<true>(v, e) : row_of<false>(v, e); };
                Edge<T> em = side(0), ec = side(1);
                Row<T> rm = row_at(above, em), rc = row_at(val[l - 1][0], ec);
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const Edge<T> ep = side(r + 2);
                    const Row<T> rp = row_at(r + 1 < R ? val[l - 1][r + 1 < R ? r + 1 : r] : below, ep);
                    const Q<T> q = WIDE && l == 1 ? inplane<true>(rm, rc, rp, em, ec, ep) : inplane<false>(rm, rc, rp, em, ec, ep);
                    rm = rc;
                    rc = rp;
                    em = ec;
                    ec = ep;
                    P3<T> f0, f1, f2;
                    fold<T>(z, q, f0, f1, f2);
                    const P3<T> ax = p3add(sa[l][r], f2);   // (A x) at plane o
                    const P3<T> xo = xp[l][r], co = cp[l][r], dd0 = dp[l][r];
                    P3<T> nv, nc = co, nd = zero3, rres = zero3;
#pragma unroll
                    for (int qq = 0; qq < 3; qq++) {
                        const T aq = comp(ax, qq);
                        T v = DELTA ? aq : comp(co, qq) + aq;
                        if (DELTA) setc(nc, qq, comp(co, qq) + v);
                        if (CHEB) {
                            const T rq = v - comp(xo, qq);
                            const T d = fmad(a.cheb[0][0][l - 1], comp(dd0, qq), a.cheb[0][1][l - 1] * rq);
                            setc(rres, qq, rq);
                            setc(nd, qq, d);
                            v = comp(xo, qq) + d;
                        }
                        setc(nv, qq, v);
                    }
                    if (l < K) {
                        const int lw = l < K ? l : 0;
                        oc[l][r] = nc;
                        od[l][r] = nd;
                        val[lw][r] = nv;
                        if (r == 0) publish(lw, pw, EDGE * w + 1, nv);
                        if (EDGE > 1 && r == R - 1) publish(lw, pw, EDGE * w + 2, nv);
                    } else if (OUT) {
                        const unsigned at = outy[r] && o < Z1 ? xout_off : DROP;
                        const unsigned sat = store ? at : DROP;
                        const size_t off = (size_t)o * plane + row[r];
#pragma unroll
                        for (int qq = 0; qq < 3; qq++) {
                            if (LAST) {
                                const T e = comp(pe[r], qq) + (DELTA ? comp(nc, qq) : comp(nv, qq));
                                buf_store(a.E[qq] + off, row_bytes, at, e);
                            } else {
                                buf_store(a.x_out[qq] + off, row_bytes, sat, comp(nv, qq));
                                if (DELTA) buf_store(a.s_out[qq] + off, row_bytes, sat, comp(nc, qq));
                                if (CHEB) buf_store(a.s_out[qq] + off, row_bytes, sat, comp(nd, qq));
                            }
                        }
                        if (resid) {
                            double s = 0.0;
#pragma unroll
                            for (int qq = 0; qq < 3; qq++) {
                                const double dd = CHEB    ? (double)comp(rres, qq)
                                                  : DELTA ? (double)comp(nv, qq)
                                                          : (double)comp(nv, qq) - (double)comp(xo, qq);
                                s += dd * dd;
                            }
                            acc += at != DROP ? s : 0.0;
                        }
                    }
                    sa[l][r] = p3add(sb[l][r], f1);
                    sb[l][r] = f0;
                    if (CHEB || l == K) xp[l][r] = P3<T>{q.X, q.Y, q.Z};
                    if (l > 1) {
                        cp[l][r] = oc[l - 1][r];
                        if (CHEB) dp[l][r] = od[l - 1][r];
                    }
                }
            }
        }
        // carried values of the plane that level 1 completes at the next step
        const size_t zc = (size_t)(zt == 0 ? nz - 1 : zt - 1) * plane;
        const bool need = t - 1 > Z0 - K && t - 1 < Z1 + K - 1;
#pragma unroll
        for (int r = 0; r < R; r++) {
            cp[1][r] = load3(cin, zc + row[r], need ? xin_off : DROP);
            if (CHEB) dp[1][r] = load3(din, zc + row[r], need ? din_off : DROP);
        }
        if (LAST) {   // E of the plane that level K completes at the next step
#pragma unroll
            for (int r = 0; r < R; r++)
                pe[r] = load3(a.E, (size_t)ze * plane + row[r], t + 1 >= tout && t + 1 < tend ? xout_off : DROP);
        }
#pragma unroll
        for (int r = 0; r < R; r++) val[0][r] = px[r];
        ev = en;
        publish(0, pw, EDGE * w + 1, px[0]);
        if (EDGE > 1) publish(0, pw, EDGE * w + 2, px[R - 1]);
        if (ring) publish(0, pw, rslot, pr);
        zt = zt + 1 == nz ? 0 : zt + 1;
        fetch(t + 1, zt);
        ze = ze + 1 == nz ? 0 : ze + 1;
        lds_barrier();
    };
    fetch(tbeg, zt);
    int t = tbeg;
    for (; t < tout; t++) step(t, std::false_type{});
    // pairs of steps let the values carried from plane to plane change their
    // registers instead of being moved (512^3 FP32: 7.5 against 7.7 ms per
    // step); the FP32 delta form, which stores twice as much, is faster
    // without (33.4 against 35.9; FP64 89.5 with, 90.9 without)
    if constexpr (DELTA && sizeof(T) == 4) {
        for (; t < tend; t++) step(t, std::true_type{});
    } else {
        for (; t < tend; t += 2) {
            step(t, std::true_type{});
            step(t + 1, std::true_type{});
        }
    }
    if (resid) {
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        __syncthreads();
        if (lane == 0) sred[w] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s_ = 0.0;
            for (int q = 0; q < NW; q++) s_ += sred[q];
            a.partial[2 * lin] = s_;
            a.partial[2 * lin + 1] = 0.0;
        }
    }
}

template <typename T>
Zc<T> zcoef(const Coef<T> &c)
{
    auto d = [](T v) { return (double)v; };
    Zc<T> z;
    z.a01 = c.a3[0][1];
    z.a02 = c.a3[0][2];
    z.o2s = (T)(d(c.o3[2]) / 6.0);
    z.o1 = c.o3[1];
    z.b00 = (T)(d(c.a3[0][0]) - 2.0 * d(c.a3[0][2]));
    z.m01 = (T)(-2.0 * d(c.a3[0][1]));
    z.o2c = (T)(d(c.o3[2]) * (4.0 / 6.0));
    z.a10 = c.a3[1][0];
    z.a12 = c.a3[1][2];
    z.o0 = c.o3[0];
    z.b11 = (T)(d(c.a3[1][1]) - 2.0 * d(c.a3[1][2]));
    z.m10 = (T)(-2.0 * d(c.a3[1][0]));
    z.a20 = c.a3[2][0];
    z.a21 = c.a3[2][1];
    z.a22 = c.a3[2][2];
    return z;
}

inline int cu_count()
{
    static std::atomic<int> cache[MX_MAX_DEVICES];
    return per_device(cache, [] {
        int dev = 0, cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu < 1)
            return 256;
        return cu;
    });
}

template <typename T, int K, int FORM, bool LAST, int R, int NW, bool WIDE>
hipError_t launch_w(const Coef<T> &c, const plan3d::Split &p, int flags, const SweepArgs<T> &a, hipStream_t s, int *nwg)
{
    static_assert(K <= plan3d::kmax(sizeof(T) == 8) && plan3d::out_x(K, WIDE) == 64 - 2 * (WIDE ? K - 1 : K));
    dim3 g(p.gx, p.gy, p.nzc);
    *nwg = g.x * g.y * g.z;
    // a workgroup leaves its partial sums in a row of its own
    if (*nwg > plan3d::partial_rows(sizeof(T) == 8, c.nx, c.ny, c.nz)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k3_stream<T, K, FORM, LAST, R, NW, WIDE>), g, dim3(64 * NW), 0, s, c, zcoef(c), a, flags, p.Lz);
    return hipGetLastError();
}

template <typename T, int K, int FORM, bool LAST, int R, int NW>
hipError_t launch_k(const Coef<T> &c, const plan3d::Split &p, int flags, const SweepArgs<T> &a, hipStream_t s, int *nwg)
{
    if (p.wide) return launch_w<T, K, FORM, LAST, R, NW, true>(c, p, flags, a, s, nwg);
    return launch_w<T, K, FORM, LAST, R, NW, false>(c, p, flags, a, s, nwg);
}

// Tiles.  Alg 1 and the delta form: two rows per wave (three or four halve the
// waves of a CU or spill: 512^3 FP32, ms per step of ten sweeps: 7.5 with 12
// waves of two rows, 8.1 with 16 of one, 8.2 with 8 of three, 8.5 with 8 of
// four), FP32 on 12 or 8 waves, FP64 on 8 or 4: the smaller one where its finer
// cut of the grid outweighs its larger rim (48 x 40 x 32 FP64: 126 against
// 153 us per step; 160 x 144 x 128 FP32: 496 against 514; 256^3 FP64 the other
// way, 4.01 against 3.84 ms).  The Chebyshev form carries half as much again
// per point and has one row per wave (512^3 FP32: 20.0 ms per step with 16
// waves, 23.6 with 8 of two rows; 160 x 144 x 128 FP64: 2.08 with 12 waves,
// 2.74 with 8 of two rows).
template <typename T, int K, int FORM, bool LAST>
hipError_t launch_shape(const Coef<T> &c, int flags, const SweepArgs<T> &a, hipStream_t s, int *nwg)
{
    constexpr bool F64 = sizeof(T) == 8, CHEB = FORM == FM_CHEB;
    if (plan3d::takes_low(F64, CHEB, K, c.nx, c.ny, c.nz)) {
        // several workgroups of the lowest tiles share a CU
        constexpr plan3d::Shape S = plan3d::low(F64, CHEB);
        return launch_k<T, K, FORM, LAST, S.r, S.nw>(c, plan3d::split(S, K, c.nx, c.ny, c.nz, 2 * cu_count()), flags, a, s, nwg);
    }
    if constexpr (CHEB) {
        constexpr plan3d::Shape S = plan3d::cheb(F64);
        return launch_k<T, K, FORM, LAST, S.r, S.nw>(c, plan3d::split(S, K, c.nx, c.ny, c.nz, cu_count()), flags, a, s, nwg);
    } else {
        constexpr plan3d::Shape SL = plan3d::large(F64), SS = plan3d::small(F64);
        const plan3d::Split l = plan3d::split(SL, K, c.nx, c.ny, c.nz, cu_count());
        const plan3d::Split m = plan3d::split(SS, K, c.nx, c.ny, c.nz, cu_count());
        if (m.cost < l.cost) return launch_k<T, K, FORM, LAST, SS.r, SS.nw>(c, m, flags, a, s, nwg);
        return launch_k<T, K, FORM, LAST, SL.r, SL.nw>(c, l, flags, a, s, nwg);
    }
}

template <typename T, int FORM, bool LAST>
hipError_t launch_form(const Coef<T> &c, int k, int flags, const SweepArgs<T> &a, hipStream_t s, int *nwg)
{
    switch (k) {
    case 1: return launch_shape<T, 1, FORM, LAST>(c, flags, a, s, nwg);
    case 2: return launch_shape<T, 2, FORM, LAST>(c, flags, a, s, nwg);
    case 3:
        if constexpr (sizeof(T) == 4) return launch_shape<T, 3, FORM, LAST>(c, flags, a, s, nwg);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

template <typename T, int FORM>
hipError_t launch_last(const Coef<T> &c, int k, int flags, const SweepArgs<T> &a, hipStream_t s, int *nwg)
{
    if (flags & SW_LAST) return launch_form<T, FORM, true>(c, k, flags, a, s, nwg);
    return launch_form<T, FORM, false>(c, k, flags, a, s, nwg);
}

}  // namespace

int stream3d_kmax(bool f64) { return plan3d::kmax(f64); }

template <typename T>
hipError_t launch_stream3d(const Coef<T> &c, int k, int form, int flags, const SweepArgs<T> &a, hipStream_t s,
                           int *nwg)
{
    if (k < 1 || k > stream3d_kmax(sizeof(T) == 8) || !plan3d::row_fits(c.nx, sizeof(T))) return hipErrorInvalidValue;
    if (form == FM_CHEB) return launch_last<T, FM_CHEB>(c, k, flags, a, s, nwg);
    if (form == FM_DELTA) return launch_last<T, FM_DELTA>(c, k, flags, a, s, nwg);
    return launch_last<T, FM_STD>(c, k, flags, a, s, nwg);
}

template hipError_t launch_stream3d<float>(const Coef<float> &, int, int, int, const SweepArgs<float> &, hipStream_t,
                                           int *);
template hipError_t launch_stream3d<double>(const Coef<double> &, int, int, int, const SweepArgs<double> &,
                                            hipStream_t, int *);

}  // namespace mx
