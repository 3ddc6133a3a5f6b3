// Vertical column work of the substep (gfx950): the interface heights, and
// the two semi-implicit column solves with everything that is per column
// around them, each in one launch.
//
// Semi-implicit column solve (riem_solver_c / riem_solver3, Sec. IX-B):
// hydrostatic interface pressure from delp (top down), nonhydrostatic
// pressure from the equation of state, interface perturbation, backward-Euler
// tridiagonal system in w (Thomas), new perturbation by a top-down scan,
// thickness by inverting the equation of state, heights by a bottom-up scan.
//
// One thread per column walking all levels is a serial chain of logarithms,
// exponentials and divisions (about 3000 cycles per level where one wavefront
// has a SIMD to itself), so a block here takes 8 to 128 columns and cuts them
// into chunks of CL consecutive layers, one thread per (column, chunk).
// Everything that is independent per layer (height transport, equation of
// state, interface coefficients, inversion) runs in all chunks at once; only
// the recurrences (pressure sum, elimination, back substitution, perturbation
// sum, height sum) pass from chunk to chunk through LDS, in the order of the
// one-thread walk, so every sum keeps its order of additions.  The layers of
// a chunk live in registers from the first load to the last store: the
// elimination coefficients, the new w and the thicknesses never go to memory.
//
// Bound by FP64 arithmetic (about 450 vector instructions per cell, two
// exponentials and three logarithms among them); memory would allow about
// 120 (site 0) and 200 us at C192 x 79.  Measured, mixed precision, against
// the launches each replaces (height update, four solve passes of one thread
// per column; thickness and commit kernels for site 1): C192 x 79 site 0
// 712 -> 384 us, site 1 712 -> 392 us; C48 x 79 (15 000 columns, fewer than
// one wavefront per SIMD before) 250 -> 40 us and 210 -> 39 us.
#include <algorithm>
#include <cmath>

#include "column.hpp"
#include "flog.hpp"
#include "launch.hpp"
#include "tridiag.hpp"

namespace fv3 {

constexpr int CNT = 256;   // threads per block

// a / c for a constant c with reciprocal rc = RN(1/c): quotient, exact
// remainder, correction (three instructions instead of the eleven of a
// general FP64 division; finite a)
DEVI double divc(double a, double c, double rc)
{
    const double q = a * rc;
    return fma(fma(-q, c, a), rc, q);
}
DEVI double div_grav(double a) { return divc(a, GRAV, 1.0 / GRAV); }
DEVI double div_pref(double a) { return divc(a, P_REF, 1.0 / P_REF); }

// Moist column solves: the equation of state takes the virtual potential
// temperature theta (1 + (Rv/Rd - 1) q), q the specific humidity (none: dry).
constexpr double RVGAS = 461.5;
constexpr double EPSV = RVGAS / RDGAS - 1.0;

// Interface value at x = 0 of the cubic whose means over four consecutive
// layers of thicknesses da, db | dc, dd (the interface between db and dc)
// are qa, qb | qc, qd: the derivative at the middle node of the quartic
// through the cumulative contents at the five layer boundaries (Lagrange
// form, contents and nodes measured from the interface).  Exact for cubics.
DEVI double cubic_iface(double da, double db, double dc, double dd, double qa, double qb, double qc, double qd)
{
    const double x0 = -(da + db), x1 = -db, x3 = dc, x4 = dc + dd;
    const double Q0 = -(qa * da + qb * db), Q1 = -qb * db, Q3 = qc * dc, Q4 = qc * dc + qd * dd;
    const double l0 = -(x1 * x3 * x4) / ((x0 - x1) * x0 * (x0 - x3) * (x0 - x4));
    const double l1 = -(x0 * x3 * x4) / ((x1 - x0) * x1 * (x1 - x3) * (x1 - x4));
    const double l3 = -(x0 * x1 * x4) / ((x3 - x0) * (x3 - x1) * x3 * (x3 - x4));
    const double l4 = -(x0 * x1 * x3) / ((x4 - x0) * (x4 - x1) * x4 * (x4 - x3));
    return Q0 * l0 + Q1 * l1 + Q3 * l3 + Q4 * l4;
}

// LDS of a column block: values a chunk hands to its neighbours
struct ColLds {
    double x[6][CNT];   // one slot per (chunk, column)
    double run[3][CNT];   // carried by the recurrence under way, one slot per column
};

// Runs f(s) for the chunks s = 0 .. nch-1 in order (UP: from the last to the
// first), each by the threads of its chunk, with what one wrote to LDS visible
// to the next.  Chunks that share a wavefront follow each other without a
// barrier (a wavefront's LDS accesses stay in order; the fence keeps the
// compiler's).
template <bool UP, class F>
DEVI void chain(int lw, int sl, int nch, F &&f)
{
    const int lg = lw < 6 ? 6 : lw, lsub = lg - lw, ng = (nch + (1 << lsub) - 1) >> lsub;
    for (int gg = 0; gg < ng; gg++) {
        const int g = UP ? ng - 1 - gg : gg;
        if (sl >> lg == g) {
            for (int q = 0; q < 1 << lsub; q++) {
                const int s = (g << lsub) + (UP ? (1 << lsub) - 1 - q : q);
                if (sl >> lw == s && s < nch) f();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
    }
}

// Address of a column's level: 32-bit byte offsets on a block-uniform base
// (SMALL: a tile's field stays below 4 GiB), or 64-bit elements.
template <bool SMALL>
struct ColOff {
    typedef long T;
};
template <>
struct ColOff<true> {
    typedef unsigned T;
};
template <bool SMALL, class T>
DEVI T &celem(T *base, typename ColOff<SMALL>::T e)
{
    if constexpr (SMALL) return *(T *)((char *)base + (size_t)(e * (unsigned)sizeof(T)));
    else return base[e];
}

// SITE 0 (riem_solver_c): half-step cells i, j in [-1, n]; the thicknesses
// are those of dz_c, the half-step interface heights by first-order upwind
// transport of the interface heights z with layer-averaged area fluxes (top
// interface: top layer), advective form, surface fixed.
// SITE 1 (riem_solver3): cells of the tile; the thicknesses are differences
// of the transported interface heights zt (FP32 deviations from zref in the
// mixed build); the transported delp, pt are committed to the state with the
// solve's w, delz and interface heights.
// EXT: the solve with options (off-centring, cubic interface perturbation,
// humidity; switched at run time), apart so that the plain one keeps its
// registers.
//
// The elimination's recurrence costs a division per level in a row; its chunk
// of layers is a fractional linear map of the ratio above it, so each chunk
// forms its 2 x 2 matrix (no division), the maps are applied chunk after chunk
// (one division per chunk), and the levels of all chunks are eliminated at once
// from there (in the form of tridiag.hpp, without cancellation).  The
// right-hand sides and the back substitution are linear maps and go the same way.
template <class B, int SITE, int CL, bool EXT, bool SMALL>
DEVI void column_body(Bk bk, const Geo &G, const MetD &M, const ColArgs<B> &A, ColLds &L)
{
    typedef typename ColOff<SMALL>::T off_t_;
    const int n = G.n, nz = G.nz, t = (int)bk.z;
    // columns per block: chunk threads of a column are CW apart
    const int CW = 1 << A.lw, sl = (int)threadIdx.x, c = sl & (CW - 1), ch = sl >> A.lw, nch = (nz + CL - 1) / CL;
    const int wdt = SITE == 0 ? n + 2 : n, p = (int)bk.x * CW + c;
    const int pc = p < wdt * wdt ? p : wdt * wdt - 1;   // idle lanes shadow the last column
    const int jr = pc / wdt, j = (SITE == 0 ? -1 : 0) + jr, i = (SITE == 0 ? -1 : 0) + (pc - jr * wdt);
    // the half-step cells form a cross (no cube corner cells)
    const bool col = p < wdt * wdt && (SITE == 1 || (i >= 0 && i < n) || (j >= 0 && j < n));
    const bool last_ch = ch == nch - 1;
    const int nx = ch >= nch - 1 ? sl : sl + CW;   // slot of the chunk below
    const int k0 = ch < nch ? ch * CL : 0;
    const bool work = ch < nch && col;
    const double kap = RDGAS / CP_AIR, gam = 1.0 / (1.0 - kap), rgam = 1.0 / gam;
    // fields: base of the tile's halo corner (block-uniform), element offset
    // of the column at the chunk's first level
    const long lev = G.lev, hb = 3 * G.pitch + 3, tb = pidx(G, nz, t, 0) - hb, tbi = pidx(G, nz + 1, t, 0) - hb;
    const unsigned pl = (unsigned)((j + 3) * (int)G.pitch + (i + 3));
    const off_t_ e0 = (off_t_)pl + (off_t_)k0 * (off_t_)lev;
    // level u of the chunk, clamped to the last one (the values of clamped
    // levels are never stored or passed on)
    auto eo = [&](int u) -> off_t_ { return k0 + u < nz ? e0 + (off_t_)u * (off_t_)lev : (off_t_)pl + (off_t_)(nz - 1) * (off_t_)lev; };
    const double dt = A.dt, dt2x = dt * dt, rdt = 1.0 / dt;
    const bool offc = EXT && A.beta != 1.0, cubic = EXT && A.cubic != 0;

    B dpi[CL], th[CL], wo[CL];
    // corner cells of the half-step grid hold nothing: neutral values there
    const bool real = SITE == 1 || (i >= 0 && i < n) || (j >= 0 && j < n);
#pragma unroll
    for (int u = 0; u < CL; u++) {
        const off_t_ o = eo(u);
        dpi[u] = celem<SMALL>(A.dpi + tb, o);
        th[u] = celem<SMALL>(A.theta + tb, o);
        wo[u] = celem<SMALL>(A.w + tb, o);
    }
    // humidity factor of the level (loaded where it is used: dry runs keep no register for it)
    auto moist = [&](int u) -> double { return EXT && A.qv ? 1.0 + EPSV * (double)celem<SMALL>(A.qv + tb, eo(u)) : 1.0; };

    // ---- layer thicknesses h (positive)
    double h[CL];
    if constexpr (SITE == 0) {
        // new heights of the interfaces above the chunk's layers
        double zn[CL];
        const double area = real ? AT(MP(M, M_AREA), i, j) : 1.0;
        // the west and east, south and north neighbours through the corner views
        auto nb = [&](int ii, int jj, int mode) -> unsigned {
            int qi = ii, qj = jj;
            bool cw;
            if (in_corner(G, SC, ii, jj)) corner_src(G, SC, ii, jj, mode, qi, qj, cw);
            return (unsigned)((qj + 3) * (int)G.pitch + (qi + 3));
        };
        const unsigned plw = nb(i - 1, j, 0), ple = nb(i + 1, j, 0), pls = nb(i, j - 1, 1), pln = nb(i, j + 1, 1);
        const unsigned P = (unsigned)G.pitch;
        const off_t_ eab = k0 > 0 ? e0 - (off_t_)lev : e0;   // layer above the chunk
        double pax0 = (double)celem<SMALL>(A.ax + tb, eab), pax1 = (double)celem<SMALL>(A.ax + tb, eab + 1);
        double pay0 = (double)celem<SMALL>(A.ay + tb, eab), pay1 = (double)celem<SMALL>(A.ay + tb, eab + P);
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const off_t_ o = eo(u), ol = o - (off_t_)pl;
            const double ax0 = (double)celem<SMALL>(A.ax + tb, o), ax1 = (double)celem<SMALL>(A.ax + tb, o + 1);
            const double ay0 = (double)celem<SMALL>(A.ay + tb, o), ay1 = (double)celem<SMALL>(A.ay + tb, o + P);
            const double zc = celem<SMALL>(A.z + tbi, o), zw = celem<SMALL>(A.z + tbi, ol + plw), ze = celem<SMALL>(A.z + tbi, ol + ple);
            const double zs = celem<SMALL>(A.z + tbi, ol + pls), zo = celem<SMALL>(A.z + tbi, ol + pln);
            const bool top = u == 0 && k0 == 0;
            const double a0 = top ? ax0 : 0.5 * (pax0 + ax0), a1 = top ? ax1 : 0.5 * (pax1 + ax1);
            const double b0 = top ? ay0 : 0.5 * (pay0 + ay0), b1 = top ? ay1 : 0.5 * (pay1 + ay1);
            const double z0 = a0 > 0 ? zw : zc, z1 = a1 > 0 ? zc : ze;
            const double y0 = b0 > 0 ? zs : zc, y1 = b1 > 0 ? zc : zo;
            zn[u] = fdiv(zc * area + a0 * z0 - a1 * z1 + b0 * y0 - b1 * y1, area + a0 - a1 + b0 - b1);
            pax0 = ax0; pax1 = ax1; pay0 = ay0; pay1 = ay1;
        }
        L.x[0][sl] = zn[0];
        __syncthreads();
        const double zbot = celem<SMALL>(A.z + tbi, (off_t_)pl + (off_t_)nz * (off_t_)lev);   // surface, fixed
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const double below = k0 + u == nz - 1 ? zbot : (u + 1 < CL ? zn[u + 1 < CL ? u + 1 : u] : L.x[0][nx]);
            h[u] = zn[u] - below;
        }
        __syncthreads();
    } else {
        // interface heights of the transported field: top of the chunk down
        auto height = [&](int u) -> double {
            const off_t_ o = eo(u);
            if constexpr (sizeof(B) == 4)
                return A.zref[t * (nz + 1) + min(k0 + u, nz - 1)] + (double)celem<SMALL>((const float *)A.zt + tbi, o);
            else return celem<SMALL>((const double *)A.zt + tbi, o);
        };
        const double surf = A.phis ? AT(A.phis + pidx(G, 1, t, 0), i, j) / GRAV : 0.0;
        double top = height(0);
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const double below = k0 + u >= nz - 1 ? surf : height(u + 1);
            // the state's thickness (negative) is below - top
            h[u] = -(below - top);
            top = below;
        }
    }

    // ---- hydrostatic interface pressure above the chunk, summed top down
    double pis = A.ptop;
    chain<false>(A.lw, sl, nch, [&]() {
        if (ch > 0) pis = L.run[0][c];
        double q = pis;
#pragma unroll
        for (int u = 0; u < CL; u++) q += (double)dpi[u];   // the last chunk's sum is not used
        L.run[0][c] = q;
    });

    // ---- equation of state: layer-mean pressure pib, perturbation pp
    double pib[CL], pp[CL];
    {
        double pi0 = pis, l0 = flog(pi0);
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const double dp = (double)dpi[u], m = div_grav(dp);
            const double pi1 = pi0 + dp, l1 = flog(pi1);
            pib[u] = fdiv(dp, l1 - l0);
            pp[u] = P_REF * fexp(gam * flog(fdiv(RDGAS * ((double)th[u] * moist(u)) * m, h[u] * P_REF))) - pib[u];
            pi0 = pi1;
            l0 = l1;
        }
    }
    // opaque, so that dpi / g and RDGAS theta are formed again where they are
    // used and not kept in registers from here to the thicknesses (with that no
    // plain instance spills; 8 to 18 registers of three of them otherwise)
#pragma unroll
    for (int u = 0; u < CL; u++) __asm__ volatile("" : "+v"(dpi[u]), "+v"(th[u]));
    // first and last layers of the chunk for its neighbours
    L.x[0][sl] = (double)dpi[0];
    L.x[1][sl] = h[0];
    L.x[2][sl] = pp[0];
    if (EXT) {
        L.x[3][sl] = (double)wo[0];
        // the cubic interface value reaches one layer further
        L.x[4][sl] = pp[1];
        L.x[5][sl] = (double)dpi[1];
    }
    __syncthreads();
    const double ndp = L.x[0][nx], nh = L.x[1][nx], npp = L.x[2][nx];
    double nw = 0.0, ndp2 = 0.0, npp2 = 0.0, pdp = 0.0, ppp = 0.0, pw = 0.0;
    if (EXT) {
        nw = L.x[3][nx];
        npp2 = L.x[4][nx];
        ndp2 = L.x[5][nx];
        __syncthreads();
        // last layer of the chunk above
        L.x[0][sl] = (double)dpi[CL - 1];
        L.x[1][sl] = pp[CL - 1];
        L.x[2][sl] = (double)wo[CL - 1];
        __syncthreads();
        if (ch > 0) {
            pdp = L.x[0][sl - CW];
            ppp = L.x[1][sl - CW];
            pw = L.x[2][sl - CW];
        }
    }
    __syncthreads();

    // ---- interface below each layer: perturbation pps, coupling Ac (pps in pp)
    const double bb = offc ? A.beta * A.beta : 1.0, ex = (1.0 - A.beta) / A.beta;
    double Ac[CL];
    {
        double pi1 = pis, ppa = ppp, dpa = pdp;   // layer above (cubic)
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const int k = k0 + u;
            const double dp0 = (double)dpi[u], dp1 = u + 1 < CL ? (double)dpi[u + 1 < CL ? u + 1 : u] : ndp;
            const double h1 = u + 1 < CL ? h[u + 1 < CL ? u + 1 : u] : nh, pp0 = pp[u], pp1 = u + 1 < CL ? pp[u + 1 < CL ? u + 1 : u] : npp;
            pi1 += dp0;
            double v;
            if (cubic && k >= 1 && k <= nz - 3) {
                const double dp2 = u + 2 < CL ? (double)dpi[u + 2 < CL ? u + 2 : u] : (u + 2 == CL ? ndp : ndp2);
                const double pp2 = u + 2 < CL ? pp[u + 2 < CL ? u + 2 : u] : (u + 2 == CL ? npp : npp2);
                v = cubic_iface(dpa, dp0, dp1, dp2, ppa, pp0, pp1, pp2);
            } else {
                v = fdiv(dp1 * pp0 + dp0 * pp1, dp0 + dp1);
            }
            const bool bottom = k == nz - 1;
            v = bottom ? pp0 : v;
            Ac[u] = fdiv(bb * gam * (pi1 + v) * dt2x, 0.5 * (bottom ? h[u] : h[u] + h1));
            ppa = pp0;
            dpa = dp0;
            pp[u] = v;
        }
    }
    L.x[0][sl] = Ac[CL - 1];
    L.x[1][sl] = pp[CL - 1];
    __syncthreads();
    const double At = ch > 0 ? L.x[0][sl - CW] : 0.0, pt_ = ch > 0 ? L.x[1][sl - CW] : 0.0;

    // ---- right-hand side (in dd); the chunk's map
    double cc[CL], dd[CL];
    ElimMap map;
#pragma unroll
    for (int u = 0; u < CL; u++) {
        const int k = k0 + u;
        const double m = div_grav((double)dpi[u]), A0 = u > 0 ? Ac[u > 0 ? u - 1 : 0] : At, p0 = u > 0 ? pp[u > 0 ? u - 1 : 0] : pt_;
        const double w0 = (double)wo[u];
        double rhs = m * w0 + dt * (pp[u] - p0);
        if (offc) {
            // P* of the interface is kept in the interface pressure's place
            // until the new perturbation is known
            if (work && k < nz) celem<SMALL>(A.pfull + tbi, eo(u) + (off_t_)lev) = pp[u];
            const double wa = k > 0 ? (u > 0 ? (double)wo[u > 0 ? u - 1 : 0] : pw) : 0.0;
            const double wb = k < nz - 1 ? (u + 1 < CL ? (double)wo[u + 1 < CL ? u + 1 : u] : nw) : 0.0;
            rhs -= ex * (Ac[u] * (w0 - wb) - A0 * (wa - w0));
        }
        dd[u] = rhs;
        map.layer(A0, Ac[u], m);
    }
    // pivot ratio above the chunk (any value at the top, where A0 is 0)
    double ein = 0.0;
    chain<false>(A.lw, sl, nch, [&]() {
        if (ch > 0) ein = L.run[1][c];
        L.run[1][c] = map(ein);
    });
    // elimination of the chunk: w_k = dd + cc w_{k+1}, dd = (part of its own
    // rows) + qq (dd above the chunk)
    double qq[CL], din = 0.0;
    {
        double dp_ = 0.0, qp = 1.0;
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const double ck = elim_layer(u > 0 ? Ac[u > 0 ? u - 1 : 0] : At, Ac[u], div_grav((double)dpi[u]), dd[u], ein, dp_, qp);
            dd[u] = dp_;
            qq[u] = qp;
            cc[u] = k0 + u < nz - 1 ? ck : 0.0;
        }
    }
    chain<false>(A.lw, sl, nch, [&]() {
        if (ch > 0) din = L.run[2][c];
        L.run[2][c] = dd[CL - 1] + qq[CL - 1] * din;
    });
#pragma unroll
    for (int u = 0; u < CL; u++) dd[u] = dd[u] + qq[u] * din;
    // ---- back substitution, bottom up (new w in dd)
    chain<true>(A.lw, sl, nch, [&]() {
        double wv = last_ch ? 0.0 : L.run[0][c];
#pragma unroll
        for (int u = CL - 1; u >= 0; u--)
            if (k0 + u < nz) {
                wv = dd[u] + cc[u] * wv;
                dd[u] = wv;
            }
        L.run[0][c] = wv;
    });
    // ---- new perturbation, top down (scan value below each layer in cc)
#pragma unroll
    for (int u = 0; u < CL; u++) cc[u] = divc(div_grav((double)dpi[u]) * (dd[u] - (double)wo[u]), dt, rdt);
    double ppt = 0.0;   // scan value above the chunk
    chain<false>(A.lw, sl, nch, [&]() {
        if (ch > 0) ppt = L.run[1][c];
        double q = ppt;
#pragma unroll
        for (int u = 0; u < CL; u++) {
            q = q + cc[u];
            cc[u] = q;
        }
        L.run[1][c] = q;
    });
    // ---- interface pressure, new thickness (in h)
    {
        const double lpref = flog(P_REF);
        double pi1 = pis;
        double pnk = ppt;
        if (offc && ch > 0) pnk = (ppt - (1.0 - A.beta) * pt_) / A.beta;
        if (work && ch == 0) celem<SMALL>(A.pfull + tbi, (off_t_)pl) = A.ptop;
#pragma unroll
        for (int u = 0; u < CL; u++) {
            const int k = k0 + u;
            const double dp = (double)dpi[u], m = div_grav(dp);
            const off_t_ o = eo(u);
            pi1 += dp;
            double pnk1 = cc[u];
            if (offc) pnk1 = (cc[u] - (1.0 - A.beta) * (work && k < nz ? celem<SMALL>(A.pfull + tbi, o + (off_t_)lev) : 0.0)) / A.beta;
            const double pn = pib[u] + 0.5 * (pnk + pnk1);
            h[u] = div_pref(RDGAS * ((double)th[u] * moist(u)) * m) * fexp(rgam * (lpref - flog(pn)));
            if (work && k < nz) {
                celem<SMALL>(A.pfull + tbi, o + (off_t_)lev) = pi1 + pnk1;
                if constexpr (SITE == 1) {
                    celem<SMALL>(A.w_out + tb, o) = (B)dd[u];
                    celem<SMALL>(A.delp_out + tb, o) = dpi[u];
                    celem<SMALL>(A.pt_out + tb, o) = th[u];
                    celem<SMALL>(A.delz_out + tb, o) = -h[u];
                }
            }
            pnk = pnk1;
        }
    }
    // ---- heights, bottom up
    chain<true>(A.lw, sl, nch, [&]() {
        double z;
        if (last_ch) {
            z = A.phis ? A.phis[pidx(G, 1, t, 0) + (long)j * G.pitch + i] / GRAV : 0.0;
            if (work) {
                const off_t_ o = (off_t_)pl + (off_t_)nz * (off_t_)lev;
                celem<SMALL>(A.phi + tbi, o) = GRAV * z;
                if constexpr (SITE == 1) celem<SMALL>(A.z_out + tbi, o) = z;
            }
        } else {
            z = L.run[2][c];
        }
#pragma unroll
        for (int u = CL - 1; u >= 0; u--)
            if (k0 + u < nz) {
                z += h[u];
                h[u] = z;
            }
        L.run[2][c] = z;
    });
#pragma unroll
    for (int u = 0; u < CL; u++) {
        if (work && k0 + u < nz) {
            celem<SMALL>(A.phi + tbi, eo(u)) = GRAV * h[u];
            if constexpr (SITE == 1) celem<SMALL>(A.z_out + tbi, eo(u)) = h[u];
        }
    }
}

template <class B, int SITE, int CL, bool EXT, bool SMALL>
DEVI void k_column(Bk bk, Geo G, MetD M, ColArgs<B> A)
{
    __shared__ ColLds L;
    column_body<B, SITE, CL, EXT, SMALL>(bk, G, M, A, L);
}
// an ensemble with a member beyond the short chunks: every member runs the
// body it runs alone
inline __host__ __device__ bool col_short(int nz, long tile) { return nz <= 160 && tile * 8 < (1L << 32); }
template <class B, int SITE, bool EXT>
DEVI void k_column_any(Bk bk, Geo G, MetD M, ColArgs<B> A)
{
    __shared__ ColLds L;
    if (col_short(G.nz, (G.nz + 1) * G.lev)) column_body<B, SITE, 5, EXT, true>(bk, G, M, A, L);
    else column_body<B, SITE, 16, true, false>(bk, G, M, A, L);
}
#define COLOCC(B, S) template <> constexpr int kocc<k_column<B, S, 5, false, true>> = 4;
COLOCC(float, 0)
COLOCC(float, 1)
COLOCC(double, 0)
COLOCC(double, 1)

// log2 of the columns per block: as many as leave a thread for every chunk,
// fewer (down to 16: one 64-byte segment of FP32) while the tiles' columns
// make fewer than two blocks per compute unit, where the idle threads cost
// nothing and the shorter blocks spread over the chip.  One chunk (up to five
// layers): 256 columns; with 128 and half the threads idle 512 x 512 x 1
// periodic takes 46 / 38 us a launch (site 0 / 1), with 256 columns 31 / 24.
static int col_shift(int chunks, long columns)
{
    int lw = 8;
    while (lw > 3 && (CNT >> lw) < chunks) lw--;
    while (lw > 4 && (columns >> lw) < 512) lw--;
    return lw;
}

template <class B, int SITE>
void column_solve(const fv3_grid *g, const ColArgs<B> &args, hipStream_t st)
{
    // Chunk length: 5 layers (up to 32 chunks).  Longer chunks hold more
    // registers: 5 layers fit the 128 a wavefront may have where four blocks
    // share a compute unit.  Beyond 160 layers, or where a tile's field
    // passes 4 GiB, chunks of 16 with 64-bit offsets (one wavefront per SIMD; two
    // substeps of a 48 x 48 x 200 cube against one thread per column, mixed / FP64
    // 4007 -> 1983 / 4893 -> 2613 us, of 24 x 24 x 512 6913 -> 1801 / 7440 -> 2401).
    const int w = SITE == 0 ? g->n + 2 : g->n;
    const bool shrt = col_short(g->nz, (long)(g->nz + 1) * g->lev);
    const int cl = shrt ? 5 : 16;
    const char *name = SITE == 0 ? "k_column_c" : "k_column_3";
    ColArgs<B> a = args;
    a.lw = col_shift((g->nz + cl - 1) / cl, (long)w * w * g->T);
    const dim3 grd((unsigned)((w * w + (1 << a.lw) - 1) >> a.lw), 1, (unsigned)g->T), blk(CNT);
    MetD M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = g->met[m];
    const bool ext = a.beta != 1.0 || a.cubic || a.qv;
    if (g_rec) {
        // one kernel serves every combination of the options, but the members of
        // an ensemble share them
        const int opts = (a.beta != 1.0 ? 1 : 0) | (a.cubic ? 2 : 0) | (a.qv ? 4 : 0);
        if (g_rec->column_options < 0) g_rec->column_options = opts;
        if (g_rec->column_options != opts) g_rec->bad = true;
    }
    if (g_rec && !g_rec->short_columns) {
        if (ext) launch_fn<k_column_any<B, SITE, true>>(name, grd, blk, st, g->geo, M, a);
        else launch_fn<k_column_any<B, SITE, false>>(name, grd, blk, st, g->geo, M, a);
    } else if (!shrt) {
        launch_fn<k_column<B, SITE, 16, true, false>>(name, grd, blk, st, g->geo, M, a);
    } else if (ext) {
        launch_fn<k_column<B, SITE, 5, true, true>>(name, grd, blk, st, g->geo, M, a);
    } else {
        launch_fn<k_column<B, SITE, 5, false, true>>(name, grd, blk, st, g->geo, M, a);
    }
}
bool column_short(const fv3_grid *g) { return col_short(g->nz, (long)(g->nz + 1) * g->lev); }
template void column_solve<float, 0>(const fv3_grid *, const ColArgs<float> &, hipStream_t);
template void column_solve<float, 1>(const fv3_grid *, const ColArgs<float> &, hipStream_t);
template void column_solve<double, 0>(const fv3_grid *, const ColArgs<double> &, hipStream_t);
template void column_solve<double, 1>(const fv3_grid *, const ColArgs<double> &, hipStream_t);

// Interface heights of the cells of a tile from the state's thicknesses,
// bottom up (once per call; each substep's second solve writes the next
// ones): the sum passes from chunk to chunk as in the solves.  Chunks of about
// five layers, 16 at most (1024 x 1024 x 2 periodic with 16 chunks whatever the
// depth 202 us, with one 16; C192 x 20 55 us, with four 22).
DEVI void k_heights(Bk bk, Geo G, int lw, int nch, const double *delz, const double *phis, double *zh)
{
    __shared__ double run[CNT];
    const int n = G.n, nz = G.nz, t = (int)bk.z;
    const int c = (int)threadIdx.x & ((1 << lw) - 1), ch = (int)threadIdx.x >> lw, p = ((int)bk.x << lw) + c;
    const bool col = p < n * n;
    const int pc = col ? p : 0, j = pc / n, i = pc % n;
    const int cl = (nz + nch - 1) / nch, k0 = ch * cl, k1 = min(nz, k0 + cl);
    const long o = (long)j * G.pitch + i, lev = G.lev;
    const double *D = delz + pidx(G, nz, t, 0) + o;
    double *Z = zh + pidx(G, nz + 1, t, 0) + o;
    constexpr int P = 8;   // loads in flight ahead of the chunk's turn
    double d[P];
#pragma unroll
    for (int u = 0; u < P; u++) d[u] = k1 - 1 - u >= k0 ? D[(long)(k1 - 1 - u) * lev] : 0.0;
    chain<true>(lw, (int)threadIdx.x, nch, [&]() {
        double z;
        if (ch == nch - 1) {
            z = phis ? phis[pidx(G, 1, t, 0) + o] / GRAV : 0.0;
            if (col) Z[(long)nz * lev] = z;
        } else {
            z = run[c];
        }
#pragma unroll
        for (int u = 0; u < P; u++)
            if (k1 - 1 - u >= k0) {
                z -= d[u];
                d[u] = z;
            }
        for (int k = k1 - 1 - P; k >= k0; k--) {
            z -= D[(long)k * lev];
            if (col) Z[(long)k * lev] = z;
        }
        run[c] = z;
    });
#pragma unroll
    for (int u = 0; u < P; u++)
        if (col && k1 - 1 - u >= k0) Z[(long)(k1 - 1 - u) * lev] = d[u];
}

void column_heights(const fv3_grid *g, const double *delz, const double *phis, double *z, hipStream_t st)
{
    const int nch = std::min(16, (g->nz + 4) / 5), lw = col_shift(nch, (long)g->n * g->n * g->T);
    launch_fn<k_heights>("k_heights", dim3((unsigned)((g->n * g->n + (1 << lw) - 1) >> lw), 1, (unsigned)g->T),
                         dim3(CNT), st, g->geo, lw, nch, delz, phis, z);
}

}  // namespace fv3
