// c_sw: the half step dt2 on the C grid, one wavefront per strip of columns,
// marching along the rows (gfx950).
//
// D -> A -> C interpolation, upwind half-step cell fluxes, kinetic energy,
// corner vorticity, C-grid winds; it writes only what later stages read: uc,
// vc, delpc, ptc, wc and the area fluxes ax, ay, on the points i, j in
// [-1, n + 1].
//
// Lane l holds column c0 - 3 + l of a strip of up to 58 columns; neighbours
// along x come from the neighbouring lanes (DPP wave shifts), those along y
// from the registers of earlier rows.  With row r the newest loaded, ua, va
// and the x faces exist on row r, the y faces on row r - 1 (va of rows r - 3
// .. r), the cells, kinetic energy and wind updates on row r - 2, the corner
// vorticity on row r - 1.  The four wavefronts of a block take four layers of
// the same strip and rows, so that the 2-D metric terms, most of the loads,
// meet in the L1 cache (the blocks of one strip dealt to one XCD gained nothing:
// 502 against 475 us).
//
// What bounds it is latency: 27 loads and stores a row with two to four
// wavefronts on a SIMD; the row of loads ahead covers most of it (metric terms
// loaded in their own row, for fewer registers: 409 against 389 us in FP32, 804
// against 713 in FP64).  C192 x 79, against tiles staged in LDS, which read
// every field (CTX + 5)(CTY + 5) / (CTX CTY) = 1.87 times and recomputed the
// face fluxes of their rims: FP32 575 -> 389 us, FP64 963 -> 713.
//
// The FP32 result is bit for bit that of the expressions as first written and
// contracted; the fma forms are therefore explicit.  FP32 with edge_interp has
// its own kernel (csw_edge.hip).
//
// Cube corner blocks are never stored.  The rows and columns that reach them
// are read through the corner views: D-grid winds and cell fields as they are
// loaded on halo rows, the A-grid winds of corner cells as the rotated
// partner component recomputed from the D-grid winds.
#include <cmath>

#include "csw.hpp"
#include "flog.hpp"
#include "launch.hpp"

#pragma clang fp contract(off)

namespace fv3 {

// One-sided stencils at cube tile edges (option edge_interp).  Along a
// sweep with tile edges at the interfaces 0 and n, the four points a, b, c,
// d are the stencil of the centred interpolation; where it would reach
// across an edge, the quadratic through the three nearest points on the own
// side (3/8, 3/4, -1/8 from the point next to the edge), and on the edge the
// mean of the two linear extrapolations of the two nearest points per side.
// cell_pt: centre of cell m from the interfaces m-1 .. m+2 (D -> A);
// face_pt: interface m from the centres m-2 .. m+1 (A -> C).
template <class B>
DEVI B centred(B a, B b, B c, B d)
{
    return (ffma((B)9, c, ffma((B)9, b, -a)) - d) * (B)0.0625;
}
template <class B>
DEVI B one_sided(B b, B c, B d)
{
    return ffma((B)-0.125, d, ffma((B)0.375, b, (B)0.75 * c));
}
template <bool EI, class B>
DEVI B cell_pt(B a, B b, B c, B d, int m, int n, bool edge)
{
    B v = centred(a, b, c, d);
    if constexpr (EI) {
        v = edge && (m == 0 || m == n) ? one_sided(b, c, d) : v;
        v = edge && (m == -1 || m == n - 1) ? one_sided(c, b, a) : v;
    }
    return v;
}
template <bool EI, class B>
DEVI B face_pt(B a, B b, B c, B d, int m, int n, bool edge)
{
    B v = centred(a, b, c, d);
    if constexpr (EI) {
        v = edge && (m == -1 || m == n - 1) ? one_sided(c, b, a) : v;
        v = edge && (m == 1 || m == n + 1) ? one_sided(b, c, d) : v;
        v = edge && (m == 0 || m == n) ? ffma((B)0.75, b + c, -((B)0.25 * (a + d))) : v;
    }
    return v;
}

// A-grid winds at a cell from the D-grid winds in memory, through the corner
// views: the sweep of ua runs along j in column i, that of va along i in row
// j; the edge rule applies on sweeps whose cross index lies inside the tile
template <bool EI, class B>
DEVI B ua_at(const Geo &G, const B *U, const B *V, int i, int j)
{
    const B a = pvx(G, U, V, SY, i, j - 1, 1, true), b = pvx(G, U, V, SY, i, j, 1, true);
    const B c = pvx(G, U, V, SY, i, j + 1, 1, true), d = pvx(G, U, V, SY, i, j + 2, 1, true);
    return cell_pt<EI>(a, b, c, d, j, G.n, i >= 0 && i < G.n);
}
template <bool EI, class B>
DEVI B va_at(const Geo &G, const B *U, const B *V, int i, int j)
{
    const B a = pvy(G, U, V, SX, i - 1, j, 0, true), b = pvy(G, U, V, SX, i, j, 0, true);
    const B c = pvy(G, U, V, SX, i + 1, j, 0, true), d = pvy(G, U, V, SX, i + 2, j, 0, true);
    return cell_pt<EI>(a, b, c, d, i, G.n, j >= 0 && j < G.n);
}

DEVI float recip(float d) { return 1.0f / d; }
DEVI double recip(double d) { return fdiv(1.0, d); }

template <class B, bool EI>
DEVI void k_csw(Bk bk, Geo G, Mets<B> M, CswArgs<B> A)
{
    constexpr unsigned SZ = sizeof(B);
    const int n = G.n, nz = G.nz, lane = (int)threadIdx.x & 63, nzb = (nz + 3) / 4;
    const int per = A.strips * A.segs, pl = (int)bk.x / per, rem = (int)bk.x - pl * per;
    const int t = pl / nzb, k = (pl - t * nzb) * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (t >= G.T || k >= nz) return;
    const int sg = rem / A.strips, sp = rem - sg * A.strips;
    // output columns c0 .. c1 - 1, rows j0 .. j1 - 1 of [-1, n + 1]
    const int c0 = -1 + sp * A.width, c1 = min(c0 + A.width, n + 2), j0 = -1 + sg * A.rows, j1 = min(j0 + A.rows, n + 2);
    if (c0 >= n + 2 || j0 >= n + 2) return;
    const int i = c0 - 3 + lane, ic = min(max(i, -3), n + 2);
    const int P = (int)G.pitch;
    const long hb = 3 * G.pitch + 3, o = pidx(G, nz, t, k) - hb, o2 = G.off0 + (long)t * G.lev - hb;
    const B *U0 = A.u + o + hb, *V0 = A.v + o + hb;   // interior origins (corner views)
    const B dt2 = A.dt2, hdt2 = (B)0.5 * dt2;
    const bool iin = i >= 0 && i < n;                                    // column inside the tile
    const bool mine = lane >= 3 && i < c1;
    const bool side = G.cube && !iin && i >= -2 && i <= n + 1;           // may be a corner cell

    struct Row {
        B u, v;                                  // U of row r + 2, V of row r
        B d, p, w, dy, py, wy;                   // cell fields of row r: x-sweep and y-sweep view
        B cu, su, dyl;                           // x faces of row r
        B cv, sv, dxl, dxc, dyc, fb, rac;        // y faces and corners of row r - 1
        B rs2, ca, ra, rdx, rdy;                 // cells and faces of row r - 2
    };
    const unsigned e0 = (unsigned)(ic + 3);
    auto row = [&](int r) -> unsigned { return ((unsigned)((min(max(r, -3), n + 2) + 3) * P) + e0) * SZ; };
    auto load = [&](int r, unsigned b, Row &R) {   // b: an opaque zero
        const unsigned br = row(r) + b, b1 = row(r - 1) + b, b2 = row(r - 2) + b;
        const unsigned bu = ((unsigned)((min(max(r + 2, -3), n + 3) + 3) * P) + e0) * SZ + b;
        R.u = el(A.u + o, bu);
        R.v = el(A.v + o, br);
        R.d = R.dy = el(A.delp + o, br);
        R.p = R.py = el(A.pt + o, br);
        R.w = R.wy = el(A.w + o, br);
        if (G.cube && (r < 0 || r >= n || r + 2 > n)) {
            // halo rows: corner points of the lanes outside the tile's columns
            const int rr = min(max(r, -3), n + 2), ru = min(max(r + 2, -3), n + 3);
            if (in_corner(G, SY, ic, ru)) R.u = pvx(G, U0, V0, SY, ic, ru, 1, true);
            if (in_corner(G, SX, ic, rr)) R.v = pvy(G, U0, V0, SX, ic, rr, 0, true);
            if (in_corner(G, SC, ic, rr)) {
                const long oo = o + hb;
                R.d = sv(G, A.delp + oo, SC, ic, rr, 0);
                R.p = sv(G, A.pt + oo, SC, ic, rr, 0);
                R.w = sv(G, A.w + oo, SC, ic, rr, 0);
                R.dy = sv(G, A.delp + oo, SC, ic, rr, 1);
                R.py = sv(G, A.pt + oo, SC, ic, rr, 1);
                R.wy = sv(G, A.w + oo, SC, ic, rr, 1);
            }
        }
        R.cu = el(M.m[M_COS_U] + o2, br);
        R.su = el(M.m[M_RSIN_U] + o2, br);
        R.dyl = el(M.m[M_DY] + o2, br);
        R.cv = el(M.m[M_COS_V] + o2, b1);
        R.sv = el(M.m[M_RSIN_V] + o2, b1);
        R.dxl = el(M.m[M_DX] + o2, b1);
        R.dxc = el(M.m[M_DXC] + o2, b1);
        R.dyc = el(M.m[M_DYC] + o2, b1);
        R.fb = el(M.m[M_FB] + o2, b1);
        R.rac = el(M.m[M_RAREA_C] + o2, b1);
        R.rs2 = el(M.m[M_RSIN2_A] + o2, b2);
        R.ca = el(M.m[M_COS_A] + o2, b2);
        R.ra = el(M.m[M_RAREA] + o2, b2);
        R.rdx = el(M.m[M_RDXC] + o2, b2);
        R.rdy = el(M.m[M_RDYC] + o2, b2);
    };

    // state: suffix 1, 2, 3 = row r - 1, r - 2, r - 3
    B um = 0, u0 = 0, u1 = 0;                      // U of rows r - 1, r, r + 1
    B uy2 = 0;                                     // U of row r - 2
    B va1 = 0, va2 = 0, va3 = 0, vb1 = 0, vb2 = 0; // va in the y-sweep view; plain (kinetic energy)
    B ua1 = 0, ua2 = 0, uc1 = 0, uc2 = 0, v1 = 0, v2 = 0;
    B d1 = 0, d2 = 0, p1 = 0, p2 = 0, w1 = 0, w2 = 0;           // cell fields, y-sweep view
    B fm1 = 0, fm2 = 0, fp1 = 0, fp2 = 0, fw1 = 0, fw2 = 0;     // x fluxes
    B gm2 = 0, gp2 = 0, gw2 = 0, vc2 = 0, ke3 = 0, vo2 = 0;
    B cu1 = 0, cu2 = 0, su1 = 0, su2 = 0, cv2 = 0, sv2 = 0, dxc2 = 0;
    const int rend = min(j1 + 2, n + 3);
    Row cur, nxt;
    unsigned zero = 0;
    load(j0 - 3, zero, cur);
    // the rows of U before the first
    auto urow = [&](int r) -> B {
        const int rr = min(max(r, -3), n + 3);
        return pvx(G, U0, V0, SY, ic, rr, 1, true);
    };
    um = urow(j0 - 4);
    u0 = urow(j0 - 3);
    u1 = urow(j0 - 2);
    for (int r = j0 - 3; r < rend; r++) {
        __asm__ volatile("" : "+v"(zero));   // addresses are formed per row, not carried in registers
        if (r + 1 < rend) load(r + 1, zero, nxt);
        // A-grid winds of row r
        const bool rin = r >= 0 && r < n;
        const B ua = cell_pt<EI>(um, u0, u1, cur.u, r, n, iin);
        const B vw = west(cur.v), ve = east(cur.v), vee = east(ve);
        const B va = cell_pt<EI>(vw, cur.v, ve, vee, i, n, rin);
        B uax = ua, vay = va;
        if (G.cube && !rin && r >= -2 && r <= n + 1) {
            if (side) {   // corner cells: the rotated partner component
                int qi, qj;
                bool cw;
                corner_src(G, SC, i, r, 0, qi, qj, cw);
                const B a = va_at<EI>(G, U0, V0, qi, qj);
                uax = cw ? -a : a;
                corner_src(G, SC, i, r, 1, qi, qj, cw);
                const B b = ua_at<EI>(G, U0, V0, qi, qj);
                vay = !cw ? -b : b;
            }
        }
        // x faces of row r
        const B uw = west(uax), uww = west(uw), ue = east(uax);
        const B uc = face_pt<EI>(uww, uw, uax, ue, i, n, rin);
        const B fl = dt2 * ffma(-cur.v, cur.cu, uc) * cur.su * cur.dyl;
        const B dw = west(cur.d), pw = west(cur.p), ww = west(cur.w);
        const bool fpos = fl > 0;
        const B fm = fl * (fpos ? dw : cur.d), fp = fm * (fpos ? pw : cur.p), fw = fm * (fpos ? ww : cur.w);
        if (mine && r >= j0 && r < j1 && r <= n && (rin ? true : i >= 0 && i <= n)) el(A.ax + o, row(r)) = fl;
        // y faces of row r - 1
        const B vc = face_pt<EI>(va3, va2, va1, vay, r - 1, n, iin);
        const B gl = dt2 * ffma(-um, cur.cv, vc) * cur.sv * cur.dxl;
        const bool gpos = gl > 0;
        const B gm = gl * (gpos ? d2 : d1), gp = gm * (gpos ? p2 : p1), gw = gm * (gpos ? w2 : w1);
        if (mine && r - 1 >= j0 && r - 1 < j1 && i <= n && (iin ? true : r - 1 >= 0 && r - 1 <= n))
            el(A.ay + o, row(r - 1)) = gl;
        // corner vorticity of row r - 1
        B ws = 1, wn = 1, wq = 1, wt = 1;   // half weights next to the missing cell at a cube vertex
        if (G.cube && (r - 1 == 0 || r - 1 == n) && (i == 0 || i == n)) {
            if (r - 1 == 0) ws = (B)0.5; else wn = (B)0.5;
            if (i == 0) wq = (B)0.5; else wt = (B)0.5;
        }
        const B vcw = west(vc), dycw = west(cur.dyc);
        const B circ = ffma(wt * vc, cur.dyc, ffma(-(wq * vcw), dycw, ffma(ws * uc2, dxc2, -(wn * uc1 * cur.dxc))));
        const B vo = ffma(circ, cur.rac, cur.fb);
        // cells of row r - 2
        const int j = r - 2;
        const bool jin = j >= 0 && j < n, jout = j >= j0 && j < j1;
        const B uce = east(uc2), fme = east(fm2), fpe = east(fp2), fwe = east(fw2);
        const B uu = ffma(-vb2, cur.ca, ua2) * cur.rs2, vv = ffma(-ua2, cur.ca, vb2) * cur.rs2;
        const B ke = hdt2 * ffma(vv, vv > 0 ? vc2 : vc, uu * (uu > 0 ? uc2 : uce));
        if (mine && jout && i <= n && j <= n && (iin || jin)) {
            const B dc = ffma(fm2 - fme + gm2 - gm, cur.ra, d2), rdc = recip(dc);
            el(A.delpc + o, row(j)) = dc;
            el(A.ptc + o, row(j)) = ffma(p2, d2, (fp2 - fpe + gp2 - gp) * cur.ra) * rdc;
            el(A.wc + o, row(j)) = ffma(w2, d2, (fw2 - fwe + gw2 - gw) * cur.ra) * rdc;
        }
        // C-grid winds of row r - 2
        const B kw = west(ke), voe = east(vo2);
        if (mine && jout) {
            if (jin && i >= 0 && i <= n) {
                const B f = dt2 * ffma(-uc2, cu2, v2) * su2;
                el(A.uc + o, row(j)) = ffma(kw - ke, cur.rdx, ffma(f, f > 0 ? vo2 : vo, uc2));
            }
            if (iin && j >= 0 && j <= n) {
                const B f = dt2 * ffma(-vc2, cv2, uy2) * sv2;
                el(A.vc + o, row(j)) = ffma(ke3 - ke, cur.rdy, ffma(-f, f > 0 ? vo2 : voe, vc2));
            }
        }
        // next row
        uy2 = um; um = u0; u0 = u1; u1 = cur.u;
        va3 = va2; va2 = va1; va1 = vay;
        vb2 = vb1; vb1 = va;
        ua2 = ua1; ua1 = ua;
        uc2 = uc1; uc1 = uc;
        v2 = v1; v1 = cur.v;
        d2 = d1; d1 = cur.dy; p2 = p1; p1 = cur.py; w2 = w1; w1 = cur.wy;
        fm2 = fm1; fm1 = fm; fp2 = fp1; fp1 = fp; fw2 = fw1; fw1 = fw;
        gm2 = gm; gp2 = gp; gw2 = gw; vc2 = vc; ke3 = ke; vo2 = vo;
        cu2 = cu1; cu1 = cur.cu; su2 = su1; su1 = cur.su; cv2 = cur.cv; sv2 = cur.sv; dxc2 = cur.dxc;
        cur = nxt;
    }
}

// FP32: 128 registers, four wavefronts per SIMD (130 and three without the
// hint: 475 against 389 us at C192 x 79)
template <> constexpr int kocc<k_csw<float, false>> = 4;

template <class B>
void csw(const fv3_grid *g, const CswArgs<B> &args, hipStream_t st)
{
    CswArgs<B> a = args;
    Mets<B> M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = sizeof(B) == 8 ? (const B *)g->met[m] : (const B *)g->metf[m];
    const int pts = g->n + 3;
    march_shape(pts, (long)g->T * ((g->nz + 3) / 4) * 4, 5, sizeof(B) == 8 ? 2 : 4, a.strips, a.width, a.segs, a.rows);
    const dim3 grd((unsigned)((long)a.strips * a.segs * g->T * ((g->nz + 3) / 4))), blk(256);
    if (g->p.edge_interp && g->p.kind == FV3_GRID_CUBED_SPHERE) {
        if constexpr (sizeof(B) == 4) csw_edge(g, a, st);
        else launch_fn<k_csw<B, true>>("k_csw", grd, blk, st, g->geo, M, a);
    } else
        launch_fn<k_csw<B, false>>("k_csw", grd, blk, st, g->geo, M, a);
}
template void csw<float>(const fv3_grid *, const CswArgs<float> &, hipStream_t);
template void csw<double>(const fv3_grid *, const CswArgs<double> &, hipStream_t);

}  // namespace fv3
