// c_sw in FP32 with one-sided stencils at cube tile edges (option edge_interp):
// one launch for the whole half step, on tiles staged in LDS.
//
// Every other c_sw marches (csw.hip).  This one keeps its tiles because its
// FP32 results are pinned: one ulp in a C-grid wind moves the FP64 fields of a
// mixed run by 1e-8, and the one-sided stencils round differently in the tiles
// with corner views and in the others, as the compiler contracts them (.375 c +
// .75 b as fma(.75, b, .375 c) or the other way round), so that a point's
// rounding depends on the tile that evaluates it.
//
// A tile of CTX x CTY points (point (i, j) = cell (i, j), its west x-face and
// south y-face, its SW corner) over i, j in [-1, n + 1] stages in LDS the
// A-grid winds (cells i0-3..i0+CTX+1), delp, pt, w (cells i0-2..i0+CTX), then
// the C-grid face quantities, the half-step kinetic energy and the corner
// vorticity, and writes only what later stages read: uc, vc, delpc, ptc, wc and
// the area fluxes ax, ay.  Each block writes the outputs of its own points.  A
// corner view's source outside the staged region is read (or, for the A-grid
// winds, recomputed) from global memory.
#include "csw.hpp"

namespace fv3 {
namespace {

typedef float B;

// Tile width: the points i in [-1, n + 1] split into ceil((n + 3) / CTX)
// tiles from i = -1; 33 covers C192's 195 points in 6 tiles (32 needed 7, the
// last with 3 useful columns: a mostly empty tile still issues every
// instruction of the kernel).
constexpr int CTX = 33, CNT = 256;
// layers per c_sw block (the block's 2-D metric terms stay in registers)
constexpr int CSL = 4;
// tile rows
constexpr int CTY = 8;

// One-sided stencils at cube tile edges (option edge_interp).  Along a
// sweep with tile edges at the interfaces 0 and n, the four points a, b, c,
// d are the stencil of the centred interpolation; where it would reach
// across an edge, the quadratic through the three nearest points on the own
// side (3/8, 3/4, -1/8 from the point next to the edge), and on the edge the
// mean of the two linear extrapolations of the two nearest points per side.
// cell_pt: centre of cell m from the interfaces m-1 .. m+2 (D -> A);
// face_pt: interface m from the centres m-2 .. m+1 (A -> C).
DEVI B cell_pt(B a, B b, B c, B d, int m, int n, bool edge)
{
    if (edge) {
        if (m == 0 || m == n) return (B)0.375 * b + (B)0.75 * c - (B)0.125 * d;
        if (m == -1 || m == n - 1) return (B)0.375 * c + (B)0.75 * b - (B)0.125 * a;
    }
    return (-a + (B)9 * b + (B)9 * c - d) / (B)16;
}
DEVI B face_pt(B a, B b, B c, B d, int m, int n, bool edge)
{
    if (edge) {
        if (m == 0 || m == n) return (B)0.75 * (b + c) - (B)0.25 * (a + d);
        if (m == 1 || m == n + 1) return (B)0.375 * b + (B)0.75 * c - (B)0.125 * d;
        if (m == -1 || m == n - 1) return (B)0.375 * c + (B)0.75 * b - (B)0.125 * a;
    }
    return (-a + (B)9 * b + (B)9 * c - d) / (B)16;
}

// the sweep of ua runs along j in column i, that of va along i in row j;
// the edge rule applies on sweeps whose cross index lies inside the tile
template <bool CORNER, bool EI>
DEVI B ua_at(const Geo &G, const B *U, const B *V, int i, int j)
{
    B a, b, c, d;
    if constexpr (CORNER) {
        a = pvx(G, U, V, SY, i, j - 1, 1, true), b = pvx(G, U, V, SY, i, j, 1, true);
        c = pvx(G, U, V, SY, i, j + 1, 1, true), d = pvx(G, U, V, SY, i, j + 2, 1, true);
    } else {
        a = AT(U, i, j - 1), b = AT(U, i, j), c = AT(U, i, j + 1), d = AT(U, i, j + 2);
    }
    return cell_pt(a, b, c, d, j, G.n, EI && i >= 0 && i < G.n);
}
template <bool CORNER, bool EI>
DEVI B va_at(const Geo &G, const B *U, const B *V, int i, int j)
{
    B a, b, c, d;
    if constexpr (CORNER) {
        a = pvy(G, U, V, SX, i - 1, j, 0, true), b = pvy(G, U, V, SX, i, j, 0, true);
        c = pvy(G, U, V, SX, i + 1, j, 0, true), d = pvy(G, U, V, SX, i + 2, j, 0, true);
    } else {
        a = AT(V, i - 1, j), b = AT(V, i, j), c = AT(V, i + 1, j), d = AT(V, i + 2, j);
    }
    return cell_pt(a, b, c, d, i, G.n, EI && j >= 0 && j < G.n);
}

// LDS elements of one c_sw block
constexpr int csw_lds()
{
    return 2 * (CTY + 5) * (CTX + 5) + 3 * (CTY + 3) * (CTX + 3) + 8 * (CTY + 2) * (CTX + 2) + 2 * (CTY + 1) * (CTX + 1);
}

// The 2-D metric terms a c_sw thread uses in phases 2-4, the same on every
// layer: loaded once per block into registers and kept for all its layers
// (the same threads own the same points on every layer).
struct CswMet {
    static constexpr int HF = CTY + 2, WF = CTX + 2, HK = CTY + 1, WK = CTX + 1;
    static constexpr int N2 = (HF * WF + CNT - 1) / CNT, N3 = (HK * WK + CNT - 1) / CNT, N4 = (CTX * CTY + CNT - 1) / CNT;
    B cu2[N2], su2[N2], dy2[N2], cv2[N2], sv2[N2], dx2[N2];                            // C-grid faces
    B rs2[N3], ca[N3], ra[N3], dxs[N3], dxn[N3], dyw[N3], dye[N3], fb[N3], rac[N3];    // cells, corners
    B cu4[N4], su4[N4], rdx4[N4], cv4[N4], sv4[N4], rdy4[N4];                          // own faces
};
DEVI void csw_metrics(const Geo &G, const Mets<B> &M, const int t, const int i0, const int j0, CswMet &Q)
{
    using Q_ = CswMet;
    constexpr int HF = Q_::HF, WF = Q_::WF, HK = Q_::HK, WK = Q_::WK;
    const int n = G.n, tid = threadIdx.x;
#pragma unroll
    for (int m = 0; m < Q_::N2; m++) {
        const int e = tid + m * CNT, r = e / WF, c = e - r * WF;
        const int i = i0 - 1 + c, j = j0 - 1 + r;
        const bool in = e < HF * WF;
        const bool xf = in && (j >= -1 && j <= n) && ((j >= 0 && j < n) ? (i >= -1 && i <= n + 1) : (i >= 0 && i <= n));
        const bool yf = in && (i >= -1 && i <= n) && ((i >= 0 && i < n) ? (j >= -1 && j <= n + 1) : (j >= 0 && j <= n));
        Q.cu2[m] = xf ? AT(MP(M, M_COS_U), i, j) : (B)0;
        Q.su2[m] = xf ? AT(MP(M, M_RSIN_U), i, j) : (B)0;
        Q.dy2[m] = xf ? AT(MP(M, M_DY), i, j) : (B)0;
        Q.cv2[m] = yf ? AT(MP(M, M_COS_V), i, j) : (B)0;
        Q.sv2[m] = yf ? AT(MP(M, M_RSIN_V), i, j) : (B)0;
        Q.dx2[m] = yf ? AT(MP(M, M_DX), i, j) : (B)0;
    }
#pragma unroll
    for (int m = 0; m < Q_::N3; m++) {
        const int e = tid + m * CNT, r = e / WK, c = e - r * WK;
        const bool in = e < HK * WK;
        // cell (i0 - 1 + c, j0 - 1 + r) of the half-step update, corner (i0 + c, j0 + r)
        const int i = i0 - 1 + c, j = j0 - 1 + r, ic = i0 + c, jc = j0 + r;
        const bool cross = in && i >= -1 && i <= n && j >= -1 && j <= n && ((i >= 0 && i < n) || (j >= 0 && j < n));
        const bool mine = cross && i >= i0 && j >= j0;
        const bool corner = in && ic >= 0 && ic <= n && jc >= 0 && jc <= n;
        Q.rs2[m] = cross ? AT(MP(M, M_RSIN2_A), i, j) : (B)0;
        Q.ca[m] = cross ? AT(MP(M, M_COS_A), i, j) : (B)0;
        Q.ra[m] = mine ? AT(MP(M, M_RAREA), i, j) : (B)0;
        Q.dxs[m] = corner ? AT(MP(M, M_DXC), ic, jc - 1) : (B)0;
        Q.dxn[m] = corner ? AT(MP(M, M_DXC), ic, jc) : (B)0;
        Q.dyw[m] = corner ? AT(MP(M, M_DYC), ic - 1, jc) : (B)0;
        Q.dye[m] = corner ? AT(MP(M, M_DYC), ic, jc) : (B)0;
        Q.fb[m] = corner ? AT(MP(M, M_FB), ic, jc) : (B)0;
        Q.rac[m] = corner ? AT(MP(M, M_RAREA_C), ic, jc) : (B)0;
    }
#pragma unroll
    for (int m = 0; m < Q_::N4; m++) {
        const int e = tid + m * CNT, r = e / CTX, c = e - r * CTX;
        const int i = i0 + c, j = j0 + r;
        const bool in = e < CTX * CTY;
        const bool fu = in && i >= 0 && i <= n && j >= 0 && j < n, fv = in && i >= 0 && i < n && j >= 0 && j <= n;
        Q.cu4[m] = fu ? AT(MP(M, M_COS_U), i, j) : (B)0;
        Q.su4[m] = fu ? AT(MP(M, M_RSIN_U), i, j) : (B)0;
        Q.rdx4[m] = fu ? AT(MP(M, M_RDXC), i, j) : (B)0;
        Q.cv4[m] = fv ? AT(MP(M, M_COS_V), i, j) : (B)0;
        Q.sv4[m] = fv ? AT(MP(M, M_RSIN_V), i, j) : (B)0;
        Q.rdy4[m] = fv ? AT(MP(M, M_RDYC), i, j) : (B)0;
    }
}

template <bool CORNER, bool EI>
DEVI void csw_body(Bk bk, B *L, const int t, const int k, const Geo &G, const CswMet &Q, B dt2, const B *u,
                   const B *v, const B *delp, const B *pt, const B *w, B *uc, B *vc, B *delpc, B *ptc, B *wc,
                   B *ax, B *ay)
{
    constexpr int WA = CTX + 5, HA = CTY + 5;   // A-grid cells i0-3.., j0-3..
    constexpr int WD = CTX + 3, HD = CTY + 3;   // delp/pt/w cells i0-2.., j0-2..
    constexpr int WF = CTX + 2, HF = CTY + 2;   // faces i0-1.., j0-1..
    constexpr int WK = CTX + 1, HK = CTY + 1;   // ke cells i0-1..; vorticity corners i0..
    B *sUA = L, *sVA = sUA + HA * WA;
    B *sD = sVA + HA * WA, *sPT = sD + HD * WD, *sW = sPT + HD * WD;
    B *sUC = sW + HD * WD, *sFm = sUC + HF * WF, *sFp = sFm + HF * WF, *sFw = sFp + HF * WF;
    B *sVC = sFw + HF * WF, *sGm = sVC + HF * WF, *sGp = sGm + HF * WF, *sGw = sGp + HF * WF;
    B *sKE = sGw + HF * WF, *sVO = sKE + HK * WK;
    const int n = G.n;
    // the thread index is made opaque per layer, so that the compiler does
    // not hoist every layer-invariant index and address of the body out of
    // the block's layer loop into registers (it then needed all 256)
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int i0 = -1 + (int)bk.x * CTX, j0 = -1 + (int)bk.y * CTY;
    const long o = pidx(G, G.nz, t, k);
    const B *U = u + o, *V = v + o, *D = delp + o, *PT = pt + o, *Wf = w + o;

    auto inA = [&](int i, int j) { return i >= i0 - 3 && i <= i0 + CTX + 1 && j >= j0 - 3 && j <= j0 + CTY + 1; };
    auto aA = [&](int i, int j) { return (j - (j0 - 3)) * WA + (i - (i0 - 3)); };
    auto inD = [&](int i, int j) { return i >= i0 - 2 && i <= i0 + CTX && j >= j0 - 2 && j <= j0 + CTY; };
    auto aD = [&](int i, int j) { return (j - (j0 - 2)) * WD + (i - (i0 - 2)); };
    auto aF = [&](int i, int j) { return (j - (j0 - 1)) * WF + (i - (i0 - 1)); };
    auto aK = [&](int i, int j) { return (j - (j0 - 1)) * WK + (i - (i0 - 1)); };
    auto aV = [&](int i, int j) { return (j - j0) * WK + (i - i0); };

    // A-grid vector through the corner view (x / y component), from LDS
    // when the source cell is staged, else recomputed from the D-grid winds
    auto UAx = [&](int i, int j, int mode) -> B {
        if (CORNER && in_corner(G, SC, i, j)) {
            int qi, qj;
            bool cw;
            corner_src(G, SC, i, j, mode, qi, qj, cw);
            B val = inA(qi, qj) ? sVA[aA(qi, qj)] : va_at<true, EI>(G, U, V, qi, qj);
            return cw ? -val : val;
        }
        return sUA[aA(i, j)];
    };
    auto VAy = [&](int i, int j, int mode) -> B {
        if (CORNER && in_corner(G, SC, i, j)) {
            int qi, qj;
            bool cw;
            corner_src(G, SC, i, j, mode, qi, qj, cw);
            B val = inA(qi, qj) ? sUA[aA(qi, qj)] : ua_at<true, EI>(G, U, V, qi, qj);
            return !cw ? -val : val;
        }
        return sVA[aA(i, j)];
    };
    // cell scalar through the corner view
    auto cv = [&](const B *sArr, const B *gArr, int i, int j, int mode) -> B {
        if (CORNER && in_corner(G, SC, i, j)) {
            int qi, qj;
            bool cw;
            corner_src(G, SC, i, j, mode, qi, qj, cw);
            return inD(qi, qj) ? sArr[aD(qi, qj)] : AT(gArr, qi, qj);
        }
        return sArr[aD(i, j)];
    };

    // 1. A-grid winds and cell scalars (corner cells are not stored)
#pragma unroll
    for (int m = 0; m < (HA * WA + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= HA * WA) break;
        int r = e / WA, c = e - r * WA;
        int i = i0 - 3 + c, j = j0 - 3 + r;
        B a = 0, b = 0;
        const bool ok = i >= -3 && i <= n + 2 && j >= -3 && j <= n + 2;
        if constexpr (CORNER) {
            if (ok && !in_corner(G, SC, i, j)) {
                if (j >= -2 && j <= n + 1) a = ua_at<CORNER, EI>(G, U, V, i, j);
                if (i >= -2 && i <= n + 1) b = va_at<CORNER, EI>(G, U, V, i, j);
            }
        } else {
            // loads at clamped points (inside the planes), then select: no
            // branches around the loads
            const bool oka = ok && j >= -2 && j <= n + 1, okb = ok && i >= -2 && i <= n + 1;
            const int ic = min(max(i, -3), n + 2), jc = min(max(j, -3), n + 2);
            a = ua_at<false, EI>(G, U, V, ic, min(max(jc, -2), n + 1));
            b = va_at<false, EI>(G, U, V, min(max(ic, -2), n + 1), jc);
            a = oka ? a : (B)0;
            b = okb ? b : (B)0;
        }
        sUA[e] = a;
        sVA[e] = b;
    }
#pragma unroll
    for (int m = 0; m < (HD * WD + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= HD * WD) break;
        int r = e / WD, c = e - r * WD;
        int i = i0 - 2 + c, j = j0 - 2 + r;
        B a = 0, b = 0, c2 = 0;
        const bool ok = i >= -3 && i <= n + 2 && j >= -3 && j <= n + 2;
        if constexpr (CORNER) {
            if (ok && !in_corner(G, SC, i, j)) {
                a = AT(D, i, j);
                b = AT(PT, i, j);
                c2 = AT(Wf, i, j);
            }
        } else {
            const int ic = min(max(i, -3), n + 2), jc = min(max(j, -3), n + 2);
            a = AT(D, ic, jc);
            b = AT(PT, ic, jc);
            c2 = AT(Wf, ic, jc);
            a = ok ? a : (B)0;
            b = ok ? b : (B)0;
            c2 = ok ? c2 : (B)0;
        }
        sD[e] = a;
        sPT[e] = b;
        sW[e] = c2;
    }
    // The D-grid winds at the faces of phases 2 and 4 are loaded one phase
    // ahead, before the barrier that ends the previous phase (the 2-D metric
    // terms of every phase are in registers for all layers of the block).
    auto xface = [&](int i, int j) {
        return (j >= -1 && j <= n) && ((j >= 0 && j < n) ? (i >= -1 && i <= n + 1) : (i >= 0 && i <= n));
    };
    auto yface = [&](int i, int j) {
        return (i >= -1 && i <= n) && ((i >= 0 && i < n) ? (j >= -1 && j <= n + 1) : (j >= 0 && j <= n));
    };
    constexpr int N2 = CswMet::N2, N4 = CswMet::N4;
    B q2V[N2], q2U[N2];
#pragma unroll
    for (int m = 0; m < N2; m++) {
        const int e = tid + m * CNT, r = e / WF, c = e - r * WF;
        const int i = i0 - 1 + c, j = j0 - 1 + r;
        const bool in = e < HF * WF, xf = in && xface(i, j), yf = in && yface(i, j);
        const int ic = min(max(i, -3), n + 2), jc = min(max(j, -3), n + 2);   // inside the planes
        const B vv = AT(V, ic, jc), uu = AT(U, ic, jc);
        q2V[m] = xf ? vv : (B)0;
        q2U[m] = yf ? uu : (B)0;
    }
    __syncthreads();
    // 2. C-grid faces: winds before the update, area fluxes, upwind fluxes
#pragma unroll
    for (int m = 0; m < (HF * WF + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= HF * WF) break;
        int r = e / WF, c = e - r * WF;
        int i = i0 - 1 + c, j = j0 - 1 + r;
        bool own = i >= i0 && i < i0 + CTX && j >= j0 && j < j0 + CTY;
        bool xf = xface(i, j), yf = yface(i, j);
        // blocks without corner views compute every face and select (all their
        // LDS reads stay inside the tile); only the global stores are masked
        B uc0 = 0, fm = 0, fp = 0, fw = 0;
        if (CORNER ? xf : true) {
            B a = UAx(i - 2, j, 0), b = UAx(i - 1, j, 0), c1 = UAx(i, j, 0), d = UAx(i + 1, j, 0);
            uc0 = face_pt(a, b, c1, d, i, n, EI && j >= 0 && j < n);
            B fl = dt2 * (uc0 - q2V[m] * Q.cu2[m]) * Q.su2[m] * Q.dy2[m];
            int up = fl > 0 ? i - 1 : i;
            fm = fl * cv(sD, D, up, j, 0);
            fp = fm * cv(sPT, PT, up, j, 0);
            fw = fm * cv(sW, Wf, up, j, 0);
            if (own && xf) AT(ax + o, i, j) = fl;
            if (!xf) uc0 = fm = fp = fw = (B)0;
        }
        sUC[e] = uc0;
        sFm[e] = fm;
        sFp[e] = fp;
        sFw[e] = fw;
        B vc0 = 0, gm = 0, gp = 0, gw = 0;
        if (CORNER ? yf : true) {
            B a = VAy(i, j - 2, 1), b = VAy(i, j - 1, 1), c1 = VAy(i, j, 1), d = VAy(i, j + 1, 1);
            vc0 = face_pt(a, b, c1, d, j, n, EI && i >= 0 && i < n);
            B fl = dt2 * (vc0 - q2U[m] * Q.cv2[m]) * Q.sv2[m] * Q.dx2[m];
            int up = fl > 0 ? j - 1 : j;
            gm = fl * cv(sD, D, i, up, 1);
            gp = gm * cv(sPT, PT, i, up, 1);
            gw = gm * cv(sW, Wf, i, up, 1);
            if (own && yf) AT(ay + o, i, j) = fl;
            if (!yf) vc0 = gm = gp = gw = (B)0;
        }
        sVC[e] = vc0;
        sGm[e] = gm;
        sGp[e] = gp;
        sGw[e] = gw;
    }
    __syncthreads();
    // 3. half-step cells (own points) and kinetic energy (one ring wider);
    //    absolute vorticity at the corners
#pragma unroll
    for (int m = 0; m < (HK * WK + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= HK * WK) break;
        int r = e / WK, c = e - r * WK;
        int i = i0 - 1 + c, j = j0 - 1 + r;
        bool cross = i >= -1 && i <= n && j >= -1 && j <= n && ((i >= 0 && i < n) || (j >= 0 && j < n));
        B kev = 0;
        if (CORNER ? cross : true) {
            B rs2 = Q.rs2[m], ca = Q.ca[m];
            B a = sUA[aA(i, j)], b = sVA[aA(i, j)];
            B uu = (a - b * ca) * rs2, vv = (b - a * ca) * rs2;
            kev = (B)0.5 * dt2 * (uu * (uu > 0 ? sUC[aF(i, j)] : sUC[aF(i + 1, j)]) +
                                  vv * (vv > 0 ? sVC[aF(i, j)] : sVC[aF(i, j + 1)]));
            if (cross && i >= i0 && j >= j0) {
                B rar = Q.ra[m];
                B dp = sD[aD(i, j)];
                B dc = dp + (sFm[aF(i, j)] - sFm[aF(i + 1, j)] + sGm[aF(i, j)] - sGm[aF(i, j + 1)]) * rar;
                B rdc = (B)1 / dc;
                AT(delpc + o, i, j) = dc;
                AT(ptc + o, i, j) =
                    (sPT[aD(i, j)] * dp + (sFp[aF(i, j)] - sFp[aF(i + 1, j)] + sGp[aF(i, j)] - sGp[aF(i, j + 1)]) * rar) * rdc;
                AT(wc + o, i, j) =
                    (sW[aD(i, j)] * dp + (sFw[aF(i, j)] - sFw[aF(i + 1, j)] + sGw[aF(i, j)] - sGw[aF(i, j + 1)]) * rar) * rdc;
            }
        }
        sKE[e] = cross ? kev : (B)0;
    }
#pragma unroll
    for (int m = 0; m < (HK * WK + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= HK * WK) break;
        int r = e / WK, c = e - r * WK;
        int i = i0 + c, j = j0 + r;
        B vo = 0;
        // outside [0, n]^2 the metric registers are zero, so vo is zero
        if (CORNER ? (i >= 0 && i <= n && j >= 0 && j <= n) : true) {
            B ws = 1, wn = 1, ww = 1, we = 1;
            if (CORNER && is_vertex(G, i, j)) {
                if (j == 0) ws = 0.5; else wn = 0.5;
                if (i == 0) ww = 0.5; else we = 0.5;
            }
            B circ = ws * sUC[aF(i, j - 1)] * Q.dxs[m] - wn * sUC[aF(i, j)] * Q.dxn[m] -
                     ww * sVC[aF(i - 1, j)] * Q.dyw[m] + we * sVC[aF(i, j)] * Q.dye[m];
            vo = Q.fb[m] + circ * Q.rac[m];
        }
        sVO[e] = vo;
    }
    B q4V[N4], q4U[N4];
#pragma unroll
    for (int m = 0; m < N4; m++) {
        const int e = tid + m * CNT, r = e / CTX, c = e - r * CTX;
        const int i = i0 + c, j = j0 + r;
        const bool in = e < CTX * CTY;
        const bool fu = in && i >= 0 && i <= n && j >= 0 && j < n, fv = in && i >= 0 && i < n && j >= 0 && j <= n;
        const int ic = min(max(i, -3), n + 2), jc = min(max(j, -3), n + 2);
        const B vv = AT(V, ic, jc), uu = AT(U, ic, jc);
        q4V[m] = fu ? vv : (B)0;
        q4U[m] = fv ? uu : (B)0;
    }
    __syncthreads();
    // 4. C-grid wind update on the interior faces of the own points
#pragma unroll
    for (int m = 0; m < (CTX * CTY + CNT - 1) / CNT; m++) {
        const int e = tid + m * CNT;
        if (e >= CTX * CTY) break;
        int r = e / CTX, c = e - r * CTX;
        int i = i0 + c, j = j0 + r;
        const bool fu = i >= 0 && i <= n && j >= 0 && j < n, fv = i >= 0 && i < n && j >= 0 && j <= n;
        if (CORNER ? fu : true) {
            B u0 = sUC[aF(i, j)];
            B fy1 = dt2 * (q4V[m] - u0 * Q.cu4[m]) * Q.su4[m];
            B vt = fy1 > 0 ? sVO[aV(i, j)] : sVO[aV(i, j + 1)];
            B un = u0 + fy1 * vt + (sKE[aK(i - 1, j)] - sKE[aK(i, j)]) * Q.rdx4[m];
            if (fu) AT(uc + o, i, j) = un;
        }
        if (CORNER ? fv : true) {
            B v0 = sVC[aF(i, j)];
            B fx1 = dt2 * (q4U[m] - v0 * Q.cv4[m]) * Q.sv4[m];
            B vt = fx1 > 0 ? sVO[aV(i, j)] : sVO[aV(i + 1, j)];
            B vn = v0 - fx1 * vt + (sKE[aK(i, j - 1)] - sKE[aK(i, j)]) * Q.rdy4[m];
            if (fv) AT(vc + o, i, j) = vn;
        }
    }
}

DEVI void k_csw_edge(Bk bk, Geo G, Mets<B> M, B dt2, const B *u, const B *v, const B *delp, const B *pt,
                const B *w, B *uc, B *vc, B *delpc, B *ptc, B *wc, B *ax, B *ay)
{
    // a block needs the corner views only if its reads (tile, staging halo
    // and the interpolation stencils around it) reach a cube corner block
    const int n = G.n;
    const int i0 = -1 + (int)bk.x * CTX, j0 = -1 + (int)bk.y * CTY;
    const bool nx = i0 - 6 < 0 || i0 + CTX + 5 > n, ny = j0 - 6 < 0 || j0 + CTY + 5 > n;
    __shared__ B L[csw_lds()];
    const int nzb = (G.nz + CSL - 1) / CSL;
    const int t = (int)bk.z / nzb, k0 = ((int)bk.z % nzb) * CSL, k1 = k0 + CSL < G.nz ? k0 + CSL : G.nz;
    CswMet Q;
    csw_metrics(G, M, t, i0, j0, Q);
    if (G.cube && nx && ny) {
#pragma clang loop unroll(disable)
        for (int k = k0; k < k1; k++)
            csw_body<true, true>(bk, L, t, k, G, Q, dt2, u, v, delp, pt, w, uc, vc, delpc, ptc, wc, ax, ay);
    } else if (nx || ny) {
#pragma clang loop unroll(disable)
        for (int k = k0; k < k1; k++)
            csw_body<false, true>(bk, L, t, k, G, Q, dt2, u, v, delp, pt, w, uc, vc, delpc, ptc, wc, ax, ay);
    } else {
#pragma clang loop unroll(disable)
        for (int k = k0; k < k1; k++)
            csw_body<false, false>(bk, L, t, k, G, Q, dt2, u, v, delp, pt, w, uc, vc, delpc, ptc, wc, ax, ay);
    }
}

}  // namespace

// six wavefronts per SIMD: 587 -> 560 us at C192 x 79 (without edge_interp)
template <> constexpr int kocc<k_csw_edge> = 6;

void csw_edge(const fv3_grid *g, const CswArgs<float> &a, hipStream_t st)
{
    Mets<float> M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = g->metf[m];
    const dim3 grd((unsigned)((g->n + 3 + CTX - 1) / CTX), (unsigned)((g->n + 3 + CTY - 1) / CTY),
                   (unsigned)(g->T * ((g->nz + CSL - 1) / CSL)));
    launch_fn<k_csw_edge>("k_csw", grd, dim3(CNT), st, g->geo, M, a.dt2, a.u, a.v, a.delp, a.pt, a.w, a.uc, a.vc,
                          a.delpc, a.ptc, a.wc, a.ax, a.ay);
}

}  // namespace fv3
