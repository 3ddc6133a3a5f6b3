// fv_tp_2d (Sec. IX-C): Lin-Rood flux-form transport on one level, one
// wavefront per strip of columns, marching along the rows (gfx950).
//
// Lane l holds column i0 - 3 + l.  The x sweeps take their neighbours from
// the neighbouring lanes (DPP wave shifts, free or one move each), the y
// sweeps carry theirs in registers from row to row: each cell's limited
// slope, edge values and parabola are computed once per sweep and used by
// both of its faces, and no value goes through LDS and no barrier is needed.
// A strip of 58 columns uses 64 lanes, a segment of R rows marches R + 6.
//
// Row r is the newest row loaded.  The outer x flux and the x-updated field
// qj exist on row r at once; the y sweeps (of the field and of qj) give the
// face between rows r - 3 and r - 2; the y-updated field qi, its x sweep and
// the cell update follow on row r - 3.
//
// MASS transports delp, pt and w together: the mass fluxes of delp weight the
// other two and its old and new values normalise them, all in registers.
// WIND turns the vorticity fluxes into the D-grid wind update.  HEIGHT
// transports the interface heights, converting them to deviations as it
// loads.  TRACER takes up to four tracers a launch.
//
// Bound by vector arithmetic (about 140 instructions per field and row of 64
// columns, 560 with everything of MASS; the tile-in-LDS kernel it replaces
// issued 488 per cell and field, its halo columns and rows counted); memory
// would allow 293 us for MASS at C192 x 79 mixed.  Measured there, per launch
// (launches replaced): MASS 835 (delp, pt, w apart) -> 435 us, WIND 336
// (vorticity fluxes, update) -> 195, HEIGHT 464 (heights, transport) -> 159,
// four tracers 1500 -> 572; FP64: 1585 -> 861, 815 -> 365, 752 -> 295.
//
// Products and sums are written as fused operations where the results are
// pinned, so that every kernel of this file rounds alike.
#include <cmath>

#include "flog.hpp"
#include "launch.hpp"
#include "march.hpp"
#include "transport.hpp"

#pragma clang fp contract(off)

namespace fv3 {

enum { MARCH_MASS = 0, MARCH_WIND = 1, MARCH_HEIGHT = 2, MARCH_TRACER = 3 };

// quotients with a shared reciprocal: FP32 by the hardware reciprocal (about
// one ulp), FP64 with Newton steps and a residual correction per quotient
DEVI float inv(float d) { return __builtin_amdgcn_rcpf(d); }
DEVI double inv(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = ffma(y, ffma(-d, y, 1.0), y);
    return ffma(y, ffma(-d, y, 1.0), y);
}
DEVI float quot(float a, float, float y) { return a * y; }
DEVI double quot(double a, double d, double y)
{
    const double q = a * y;
    return ffma(ffma(-d, q, a), y, q);
}

// limited slope of order 8 (zero at an extremum), plain slope otherwise
template <int ORD, class T>
DEVI T slope(T a, T b, T c)
{
    const T d = (c - a) * (T)0.25;
    if constexpr (ORD != 8) return d;
    const T mx = fmax(a, fmax(b, c)), mn = fmin(a, fmin(b, c));
    return copysign(fmin(fabs(d), fmin(mx - b, b - mn)), d);
}
// fourth-order edge value between cells a and b with slopes da, db
template <class T>
DEVI T edge(T a, T b, T da, T db)
{
    return ffma((T)0.5, a + b, (da - db) * ((T)1 / (T)3));
}
// edge deviations of cell q (slope dm, edge values al, ar)
template <int ORD, class T>
DEVI void parabola(T q, T dm, T al, T ar, bool flat, T &bl, T &br)
{
    bl = al - q;
    br = ar - q;
    if constexpr (ORD == 8) {
        const T a2 = (T)2 * fabs(dm);
        bl = copysign(fmin(a2, fabs(bl)), -dm);
        br = copysign(fmin(a2, fabs(br)), dm);
    }
    if constexpr (ORD == 5) {
        // 2dx-filtered: the cell mean alone
        bl = flat ? (T)0 : bl;
        br = flat ? (T)0 : br;
    }
    if constexpr (ORD == 7) {
        // positive-definite: the parabola of a cell of non-negative mean is
        // scaled about the mean until its minimum over the cell is zero
        if (q >= (T)0) {
            const T aL = q + bl, aR = q + br, a6 = (T)-3 * (bl + br), da = aR - aL;
            T mn = fmin(aL, aR);
            if (a6 < (T)0 && fabs(da) < -a6) mn = fmin(mn, q + da * da / ((T)4 * a6) + a6 / (T)12);
            if (mn < (T)0) {
                const T th = q / (q - mn);
                bl *= th;
                br *= th;
            }
        }
    }
}
// swept mean of the upwind cell: q + (1 - |c|) (e - |c| s), e the deviation
// of the swept edge, s the sum of both
template <class T>
DEVI T swept(T q, T e, T s, T c)
{
    const T cc = fabs(c);
    return ffma((T)1 - cc, ffma(-cc, s, e), q);
}

// face value between columns i - 1 and i from one row's cells
template <int ORD, class T>
DEVI T xface(T q, T c)
{
    const T qw = west(q), qe = east(q), dm = slope<ORD>(qw, q, qe);
    const T al = edge(qw, q, west(dm), dm), ar = east(al);
    bool flat = false;
    if constexpr (ORD == 5) {
        // both the cell and a neighbour are strict local extrema
        const T x = (q - qw) * (qe - q) < (T)0 ? (T)1 : (T)0, xw = west(x), xe = east(x);
        flat = x != (T)0 && (xw != (T)0 || xe != (T)0);
    }
    T bl, br;
    parabola<ORD>(q, dm, al, ar, flat, bl, br);
    // every lane takes part in a shift: none inside a conditional
    const T s = bl + br, brw = west(br), sw = west(s);
    const bool pos = c > 0;
    return swept(pos ? qw : q, pos ? brw : bl, pos ? sw : s, c);
}

// the same along y: push(x, c) takes row r and returns the face between rows
// r - 3 and r - 2 for its Courant number c
template <int ORD, class T>
struct YSweep {
    T q1 = 0, q2 = 0, q3 = 0, dm2 = 0, al2 = 0, br3 = 0, s3 = 0;
    bool x2 = false, x3 = false;
    DEVI T push(T x, T c)
    {
        const T dm1 = slope<ORD>(q2, q1, x), al1 = edge(q2, q1, dm2, dm1);
        bool x1 = false, flat = false;
        if constexpr (ORD == 5) {
            x1 = (q1 - q2) * (x - q1) < (T)0;
            flat = x2 && (x3 || x1);
        }
        T bl, br;
        parabola<ORD>(q2, dm2, al2, al1, flat, bl, br);
        const T s = bl + br;
        const bool pos = c > 0;
        const T f = swept(pos ? q3 : q2, pos ? br3 : bl, pos ? s3 : s, c);
        q3 = q2;
        br3 = br;
        s3 = s;
        q2 = q1;
        q1 = x;
        dm2 = dm1;
        al2 = al1;
        x3 = x2;
        x2 = x1;
        return f;
    }
};

template <class T, int KIND, int NF, int ORD>
DEVI void k_march(Bk bk, Geo G, MarchArgs<T> A)
{
    constexpr unsigned SZ = sizeof(T);
    // rows per turn of the loop: three keep the rows' values from moving between
    // registers, which pays where one field's state leaves room for them
    constexpr int UNR = NF == 1 ? 3 : 1;
    const int n = G.n, nz = G.nz, lane = (int)threadIdx.x & 63;
    // one unit (plane, segment, strip) per wavefront
    const int unit = __builtin_amdgcn_readfirstlane((int)bk.x * 4 + ((int)threadIdx.x >> 6));
    const int per = A.strips * A.segs;
    const int pl = unit / per, rem = unit - pl * per, sg = rem / A.strips, sp = rem - sg * A.strips;
    if (pl >= G.T * nz) return;
    const int t = pl / nz, k = pl - t * nz;
    const int i0 = sp * A.width, i1 = min(i0 + A.width, n), j0 = sg * A.rows, j1 = min(j0 + A.rows, n);
    if (j0 >= n || i0 >= n) return;
    const int i = i0 - 3 + lane, ic = min(i, n + 2);   // columns past the halo repeat the last one
    const int P = (int)G.pitch;
    const int Lq = KIND == MARCH_HEIGHT ? nz + 1 : nz;
    // halo corners of the planes (block-uniform); elements of a plane are
    // addressed by 32-bit byte offsets from there
    const long hb = 3 * G.pitch + 3;
    const long oq = pidx(G, Lq, t, k) - hb, oc = pidx(G, nz, t, k) - hb, o2 = G.off0 + (long)t * G.lev - hb;
    const bool avg = KIND == MARCH_HEIGHT && k > 0;   // interface: mean of layers k - 1 and k
    const long ocb = avg ? oc - G.lev : oc;
    const double zr = KIND == MARCH_HEIGHT && sizeof(T) == 4 ? A.z[oq + hb] : 0.0;
    if constexpr (KIND == MARCH_HEIGHT && sizeof(T) == 4) {
        if (rem == 0 && lane == 0) A.zref[t * (nz + 1) + k] = zr;
    }

    // one row as loaded (conversions wait until the row is used, so that its
    // loads stay in flight): the field in the x-sweep and the y-sweep view,
    // x faces of row r, y faces of row r - 2, the upper layer's for averages
    constexpr int NA = KIND == MARCH_HEIGHT ? 2 : 1;
    using Q = typename std::conditional<KIND == MARCH_HEIGHT, double, T>::type;
    struct Row {
        Q q[NF], qy[NF];
        T crx[NA], xfx[NA], cry[NA], yfx[NA], ar;
    };
    // element e of the plane of field f
    auto field = [&](int f, unsigned e) -> Q {
        if constexpr (KIND == MARCH_HEIGHT) return el(A.z + oq, e * 8u);
        else return el(A.q[f] + oq, e * SZ);
    };
    // FP32 heights travel as deviations from the plane's reference
    auto value = [&](Q q) -> T { return KIND == MARCH_HEIGHT && SZ == 4 ? (T)(q - zr) : (T)q; };
    auto mean = [&](const T *c) -> T { return KIND == MARCH_HEIGHT && avg ? (T)0.5 * (c[NA - 1] + c[0]) : c[0]; };
    const unsigned ei = (unsigned)(ic + 3);
    // row r (element offset er of its column ic), faces of row r - 2 at ev
    auto load = [&](int r, unsigned er, unsigned ev, Row &R) {
        const bool halo_row = G.cube && (r < 0 || r >= n);   // its ends are cube corner cells
        if (!halo_row) {
#pragma unroll
            for (int f = 0; f < NF; f++) R.q[f] = R.qy[f] = field(f, er);
        } else {
            unsigned ex = er, ey = er;
            if (in_corner(G, SC, ic, r)) {
                int xi, xj, yi, yj;
                bool cw;
                corner_src(G, SC, ic, r, 0, xi, xj, cw);
                corner_src(G, SC, ic, r, 1, yi, yj, cw);
                ex = (unsigned)((xj + 3) * P + xi + 3);
                ey = (unsigned)((yj + 3) * P + yi + 3);
            }
#pragma unroll
            for (int f = 0; f < NF; f++) {
                R.q[f] = field(f, ex);
                R.qy[f] = field(f, ey);
            }
        }
        const unsigned br = er * SZ, bv = ev * SZ;
        R.crx[0] = el(A.crx + oc, br);
        R.xfx[0] = el(A.xfx + oc, br);
        R.cry[0] = el(A.cry + oc, bv);
        R.yfx[0] = el(A.yfx + oc, bv);
        R.ar = el(A.area + o2, br);
        if constexpr (KIND == MARCH_HEIGHT) {
            R.crx[NA - 1] = el(A.crx + ocb, br);
            R.xfx[NA - 1] = el(A.xfx + ocb, br);
            R.cry[NA - 1] = el(A.cry + ocb, bv);
            R.yfx[NA - 1] = el(A.yfx + ocb, bv);
        }
    };

    YSweep<ORD, T> Y[NF], Yj[NF];
    // delay lines: rows r - 1, r - 2, r - 3 of the outer x flux, the x Courant
    // numbers and fluxes and the area; the previous y face (the field's rows
    // are in its y sweep)
    T fx[NF][3] = {}, crxd[3] = {}, xfxd[3] = {}, ard[3] = {};
    T fyp[NF] = {}, Fyp[NF] = {}, yfp = 0, kep = 0;
    double myp = 0.0;
    (void)kep;
    (void)myp;
    const bool cell = lane >= 3 && i < i1;                             // cells of the strip
    const bool xown = lane >= 3 && (i < i1 || (i == i1 && i1 == n));   // x faces it owns

    Row cur, nxt;
    // element offsets of the rows r (newest), v (y faces, r - 2) and u (cells, r - 3)
    unsigned er = (unsigned)(j0 * P) + ei, ev = er + 3u * (unsigned)P, eu = ev;
    load(j0 - 3, er, ev, cur);
    auto step = [&](int r) {
        // opaque per row, so that no per-array address is carried in vector
        // registers from row to row
        __asm__ volatile("" : "+v"(er), "+v"(ev), "+v"(eu));
        const bool upd = r - 3 >= j0;                                   // row r - 3 is a row of the segment
        const int rv = r - 2;
        const bool yown = rv >= j0 && (rv < j1 || rv == n);             // y faces of row r - 2
        const unsigned ou = eu * SZ, ov = ev * SZ, odu = eu * 8u, odv = ev * 8u;
        // operands of this row's epilogue and the next row, ahead of the arithmetic
        double amx = 0, amy = 0, mx = 0, my = 0, pa = 0, pb = 0, a64 = 1;
        (void)pb;
        T acx = 0, acy = 0, ke = 0, un = 0, vn = 0, rdx = 0, rdy = 0;
        if constexpr (KIND == MARCH_MASS) {
            amx = el(A.mfx + oc, odu);
            acx = el(A.cxa + oc, ou);
            amy = el(A.mfy + oc, odv);
            acy = el(A.cya + oc, ov);
        }
        if constexpr (KIND == MARCH_TRACER) {
            mx = el(A.mx + oc, odu);
            my = el(A.my + oc, odv);
            pa = el(A.dp1 + oc, odu);
            a64 = el(A.area64 + o2, odu);
        }
        if constexpr (KIND == MARCH_WIND) {
            ke = el(A.ke + oc, ov);
            un = el(A.u + oc, ov);
            vn = el(A.v + oc, ou);
            rdx = el(A.rdx + o2, ov);
            rdy = el(A.rdy + o2, ou);
        }
        er += (unsigned)P;
        if (r + 1 < j1 + 3) load(r + 1, er, rv >= j0 ? ev + (unsigned)P : ev, nxt);

        const T crx = mean(cur.crx), xfx = mean(cur.xfx), cry = mean(cur.cry), yfx = mean(cur.yfx);
        // outer x sweep and x-updated field on row r; y sweeps to face r - 2
        const T xfe = east(xfx), dx = cur.ar + xfx - xfe, rx = inv(dx);
        const T dy = ard[2] + yfp - yfx, ry = inv(dy);
        T fxn[NF], fy[NF], Fy[NF], qu[NF];
        T wy = yfx;
        if constexpr (KIND == MARCH_TRACER) {
            // mass fluxes of one sub-cycle; the layer mass after it
            mx = ffma(ffma(-(mx * A.rrs), A.rs, mx), A.rrs, mx * A.rrs);
            my = ffma(ffma(-(my * A.rrs), A.rs, my), A.rrs, my * A.rrs);
            wy = (T)my;
            if (upd) {
                pb = pa + fdiv(mx - east(mx) + myp - my, a64);
                if (A.dp2 && cell) el(A.dp2 + oc, odu) = pb;
            }
            myp = my;
        }
#pragma unroll
        for (int f = 0; f < NF; f++) {
            const T q = value(cur.q[f]);
            fxn[f] = xface<ORD>(q, crx);
            const T qj = quot(ffma(-xfe, east(fxn[f]), ffma(q, cur.ar, xfx * fxn[f])), dx, rx);
            qu[f] = Y[f].q3;   // row r - 3
            fy[f] = Y[f].push(value(cur.qy[f]), cry);
            const T fyj = Yj[f].push(qj, cry);
            Fy[f] = (T)0.5 * (fyj + fy[f]) * (KIND == MARCH_MASS && f > 0 ? Fy[0] : wy);
        }
        if (upd) {
            // y-updated field, its x sweep, final x flux and the cells of row r - 3
            T Fx[NF], dold = 0, dnew = 0;
            const T xf3 = xfxd[2], ar3 = ard[2];
#pragma unroll
            for (int f = 0; f < NF; f++) {
                const T q3 = qu[f];
                const T qi = quot(ffma(-yfx, fy[f], ffma(q3, ar3, yfp * fyp[f])), dy, ry);
                const T fxi = xface<ORD>(qi, crxd[2]);
                const T wx = KIND == MARCH_MASS && f > 0 ? Fx[0] : KIND == MARCH_TRACER ? (T)mx : xf3;
                Fx[f] = (T)0.5 * (fxi + fx[f][2]) * wx;
                const T fe = east(Fx[f]);
                T out = 0;
                if constexpr (KIND == MARCH_MASS) {
                    if (f == 0) {
                        const T num = Fx[f] - fe + Fyp[f] - Fy[f];
                        if constexpr (sizeof(T) == 4) out = ffma(inv(ar3), num, q3);
                        else out = q3 + quot(num, ar3, inv(ar3));
                        dold = q3;
                        dnew = out;
                    } else {
                        const T d = dnew * ar3;
                        out = quot(ffma(ar3, q3 * dold, Fx[f]) - fe + Fyp[f] - Fy[f], d, inv(d));
                    }
                } else if constexpr (KIND == MARCH_HEIGHT) {
                    const T d = ar3 + xf3 - east(xf3) + yfp - yfx;
                    out = quot(ffma(q3, ar3, Fx[f]) - fe + Fyp[f] - Fy[f], d, inv(d));
                } else if constexpr (KIND == MARCH_TRACER) {
                    const double a = (double)ar3;
                    out = (T)fdiv(ffma((double)q3 * pa, a, (double)Fx[f]) - (double)fe + (double)Fyp[f] - (double)Fy[f], pb * a);
                }
                if constexpr (KIND != MARCH_WIND) {
                    if (cell) el(A.out[f] + oq, ou) = out;
                }
                if constexpr (KIND == MARCH_MASS) {
                    if (f == 0 && xown) {
                        el(A.mfx + oc, odu) = amx + (double)Fx[0];
                        el(A.cxa + oc, ou) = acx + crxd[2];
                    }
                }
                if constexpr (KIND == MARCH_MASS || KIND == MARCH_TRACER) {
                    if (A.FX[f] && xown && (i == 0 || i == n)) el(A.FX[f] + oc, ou) = Fx[f];
                }
            }
            if constexpr (KIND == MARCH_WIND) {
                // v on x face (i, r - 3): kinetic energy of rows r - 3 and r - 2
                T dv = 0;
                if (A.nuv > (T)0) {
                    const T wc = qu[0] - el(A.fc + o2, ou), ww = west(wc);
                    dv = -A.nuv * (ww - wc) * el(A.rdxc + o2, ou);
                }
                if (xown) el(A.v + oc, ou) = ffma(kep - ke - Fx[0], rdy, vn) + dv;
            }
        }
        if constexpr (KIND == MARCH_MASS) {
            if (yown && cell) {
                el(A.mfy + oc, odv) = amy + (double)Fy[0];
                el(A.cya + oc, ov) = acy + cry;
            }
        }
        if constexpr (KIND == MARCH_MASS || KIND == MARCH_TRACER) {
            if (yown && cell && (rv == 0 || rv == n)) {
#pragma unroll
                for (int f = 0; f < NF; f++)
                    if (A.FY[f]) el(A.FY[f] + oc, ov) = Fy[f];
            }
        }
        if constexpr (KIND == MARCH_WIND) {
            const T kee = east(ke);
            if (yown) {
                T du = 0;
                if (A.nuv > (T)0) {
                    const T wc = Y[0].q3 - el(A.fc + o2, ov), ws = qu[0] - el(A.fc + o2, ov - (unsigned)P * SZ);
                    du = A.nuv * (ws - wc) * el(A.rdyc + o2, ov);
                }
                if (cell) el(A.u + oc, ov) = ffma(ke - kee + Fy[0], rdx, un) + du;
            }
            kep = ke;
        }
        // shift the delay lines
#pragma unroll
        for (int f = 0; f < NF; f++) {
            fx[f][2] = fx[f][1];
            fx[f][1] = fx[f][0];
            fx[f][0] = fxn[f];
            fyp[f] = fy[f];
            Fyp[f] = Fy[f];
        }
        crxd[2] = crxd[1]; crxd[1] = crxd[0]; crxd[0] = crx;
        xfxd[2] = xfxd[1]; xfxd[1] = xfxd[0]; xfxd[0] = xfx;
        ard[2] = ard[1]; ard[1] = ard[0]; ard[0] = cur.ar;
        yfp = yfx;
        if (rv >= j0) ev += (unsigned)P;
        if (upd) eu += (unsigned)P;
        cur = nxt;
    };
    for (int r = j0 - 3, end = j1 + 3;;) {
        step(r);
        if (++r == end) break;
        if constexpr (UNR == 3) {
            step(r);
            if (++r == end) break;
            step(r);
            if (++r == end) break;
        }
    }
}

// FP32 MASS: 128 registers (4 to 8 of them spilled), four wavefronts per SIMD
// (132 and three without the hint: 479 against 471 us at C192 x 79); FP64 MASS:
// 256, two
#define MARCHOCC(T, ORD, W) template <> constexpr int kocc<k_march<T, MARCH_MASS, 3, ORD>> = W;
MARCHOCC(float, 8, 4)
MARCHOCC(float, 6, 4)
MARCHOCC(float, 5, 4)
MARCHOCC(double, 8, 2)
MARCHOCC(double, 6, 2)
MARCHOCC(double, 5, 2)

// wavefronts per SIMD of each kernel, from its registers (orders 5, 7 and 8; of
// order 6 FP32 HEIGHT fits seven, one FP32 tracer seven, one FP64 tracer four)
template <int KIND, int NF, class T>
constexpr int march_occ()
{
    if (sizeof(T) == 8) return NF == 1 ? 3 : 2;
    return KIND == MARCH_TRACER ? (NF == 1 ? 5 : NF == 2 ? 4 : 3) : KIND == MARCH_MASS ? 4 : 6;
}

template <class T>
static unsigned transport_shape(const fv3_grid *g, MarchArgs<T> &a, int occ)
{
    const long planes = (long)g->T * g->nz;
    march_shape(g->n, planes, 6, occ, a.strips, a.width, a.segs, a.rows);
    return (unsigned)((planes * a.strips * a.segs + 3) / 4);
}

template <int KIND, int NF, class T>
static void march(const char *name, const fv3_grid *g, int ord, MarchArgs<T> a, hipStream_t st)
{
    const dim3 grd(transport_shape(g, a, march_occ<KIND, NF, T>())), blk(256);
    if (ord == 5) launch_fn<k_march<T, KIND, NF, 5>>(name, grd, blk, st, g->geo, a);
    else if (ord == 6) launch_fn<k_march<T, KIND, NF, 6>>(name, grd, blk, st, g->geo, a);
    else launch_fn<k_march<T, KIND, NF, 8>>(name, grd, blk, st, g->geo, a);
}

template <class T>
void march_mass(const fv3_grid *g, MarchArgs<T> a, hipStream_t st)
{
    march<MARCH_MASS, 3>("k_march_mass", g, g->p.hord, a, st);
}
template <class T>
void march_wind(const fv3_grid *g, MarchArgs<T> a, hipStream_t st)
{
    march<MARCH_WIND, 1>("k_march_wind", g, g->p.hord, a, st);
}
template <class T>
void march_height(const fv3_grid *g, MarchArgs<T> a, hipStream_t st)
{
    march<MARCH_HEIGHT, 1>("k_march_height", g, g->p.hord, a, st);
}

template <int NF, class T>
static void march_tracer_n(const fv3_grid *g, const MarchArgs<T> &a, hipStream_t st)
{
    const int ord = g->p.hord_tr ? g->p.hord_tr : g->p.hord;
    MarchArgs<T> b = a;
    const dim3 grd(transport_shape(g, b, march_occ<MARCH_TRACER, NF, T>())), blk(256);
    if (ord == 7) launch_fn<k_march<T, MARCH_TRACER, NF, 7>>("k_march_tracer", grd, blk, st, g->geo, b);
    else march<MARCH_TRACER, NF>("k_march_tracer", g, ord, a, st);
}
template <class T>
void march_tracer(const fv3_grid *g, int nq, MarchArgs<T> a, hipStream_t st)
{
    a.rrs = 1.0 / a.rs;
    if (nq == 1) march_tracer_n<1>(g, a, st);
    else if (nq == 2) march_tracer_n<2>(g, a, st);
    else if (nq == 3) march_tracer_n<3>(g, a, st);
    else if constexpr (sizeof(T) == 4) march_tracer_n<4>(g, a, st);
}

#define MARCH_INST(T)                                                        \
    template void march_mass<T>(const fv3_grid *, MarchArgs<T>, hipStream_t); \
    template void march_wind<T>(const fv3_grid *, MarchArgs<T>, hipStream_t); \
    template void march_height<T>(const fv3_grid *, MarchArgs<T>, hipStream_t); \
    template void march_tracer<T>(const fv3_grid *, int, MarchArgs<T>, hipStream_t);
MARCH_INST(float)
MARCH_INST(double)

}  // namespace fv3
