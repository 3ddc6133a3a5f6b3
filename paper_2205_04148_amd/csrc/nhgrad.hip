// nh_p_grad: corner values by the fourth-order (-1, 7, 7, -1)/12 tensor
// interpolation of pfull and phi at a layer's two interfaces and of delp, then
// the finite-volume pressure gradient along each D-grid edge; one wavefront
// per strip of columns and NL layers, marching along the rows (gfx950).
//
// Lane l holds column c0 - 2 + l of a strip of up to 58 corners.  The x pass of
// a row takes its neighbours from the neighbouring lanes (DPP wave shifts), the
// y pass from the registers of the three rows before: with row r the newest
// loaded, the corners of row r - 1 exist, u is updated on row r - 1 and v,
// between two corner rows, on row r - 2.  The four wavefronts of a block take
// consecutive layers of one strip, whose shared interfaces meet in the L1
// cache.
//
// Bound by vector arithmetic: per row and layer 5 fields of two 4-tap passes
// and two gradients; with two layers a wavefront the interface between them is
// interpolated once (8 fields for two layers).  C192 x 79, against corner tiles
// interpolated in LDS with five barriers a layer: 298 -> 203 us mixed, 301 -> 266
// FP64; C48 x 79 mixed 37.6 -> 24.5; periodic 48 x 8 18.5 -> 6.2 (its blocks walked
// eight layers one after the other).
//
// Cells of cube corner blocks are read through the x-sweep corner view on the
// halo rows; a corner at a cube vertex is the mean of its three cells.
#include <cmath>

#include "flog.hpp"
#include "launch.hpp"
#include "nhgrad.hpp"

#pragma clang fp contract(off)

namespace fv3 {

// cell means x0..x3 of the cells m-2 .. m+1 to interface m: (-1,7,7,-1)/12,
// or with `edge` next to a tile edge (interfaces 0, n) the interface value
// of the quadratic with the three nearest cell means on the own side
// (1/3, 5/6, -1/6), on the edge the mean of the two sides' linear
// extrapolations (option edge_interp)
template <bool EI>
DEVI double face_mean(double x0, double x1, double x2, double x3, int m, int n, bool edge)
{
    constexpr double W0 = -1.0 / 12.0, W1 = 7.0 / 12.0;
    double r = ffma(W0, x3, ffma(W1, x2, ffma(W1, x1, W0 * x0)));
    if constexpr (EI) {
        if (edge && (m == -1 || m == n - 1)) r = fdiv(ffma(2.0, x2, 5.0 * x1) - x0, 6.0);
        if (edge && (m == 1 || m == n + 1)) r = fdiv(ffma(2.0, x1, 5.0 * x2) - x3, 6.0);
        if (edge && (m == 0 || m == n)) r = ffma(0.75, x1 + x2, -(0.25 * (x0 + x3)));
    }
    return r;
}

// Finite-volume pressure gradient between two columns W, E over one layer:
// contour integral of p dPhi around the quadrilateral of the two columns'
// interfaces, over the mean layer mass and the distance L.
DEVI double layer_pgf(double dt, double L, double dW, double dE, double zW0, double zW1, double zE0, double zE1,
                      double pW0, double pW1, double pE0, double pE1)
{
    return fdiv(dt, L * (dW + dE)) * ffma(zW0 - zE1, pW1 - pE0, (zW1 - zE0) * (pE1 - pW0));
}

template <class B, bool EI, int NL>
DEVI void nhpgrad_body(Bk bk, const Geo &G, const MetD &M, const NhArgs<B> &A)
{
    // fields: p at NL + 1 interfaces, phi at NL + 1, delp of NL layers
    constexpr int NI = NL + 1, NF = 2 * NI + NL;
    const int n = G.n, nz = G.nz, lane = (int)threadIdx.x & 63, nzb = (nz + 4 * NL - 1) / (4 * NL);
    const int per = A.strips * A.segs, pl = (int)bk.x / per, rem = (int)bk.x - pl * per;
    const int t = pl / nzb, k = ((pl - t * nzb) * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * NL;
    if (t >= G.T || k >= nz) return;
    const int sg = rem / A.strips, sp = rem - sg * A.strips;
    // corner columns c0 .. c1 - 1 and rows j0 .. j1 - 1 of [0, n]
    const int c0 = sp * A.width, c1 = min(c0 + A.width, n + 1), j0 = sg * A.rows, j1 = min(j0 + A.rows, n + 1);
    if (c0 > n || j0 > n) return;
    const int i = c0 - 2 + lane, ic = min(i, n + 2), P = (int)G.pitch;
    const long hb = 3 * G.pitch + 3;
    const bool mine = lane >= 2 && i < c1, fu = mine && i < n;
    long oi[NI], ol[NL];
#pragma unroll
    for (int q = 0; q < NI; q++) oi[q] = pidx(G, nz + 1, t, min(k + q, nz)) - hb;
#pragma unroll
    for (int q = 0; q < NL; q++) ol[q] = pidx(G, nz, t, min(k + q, nz - 1)) - hb;
    const long o2 = G.off0 + (long)t * G.lev - hb;
    const unsigned e0 = (unsigned)(ic + 3);
    auto row = [&](int r) -> unsigned { return (unsigned)(min(max(r, -3), n + 2) + 3) * (unsigned)P + e0; };
    struct Row {
        double p[NI], z[NI];
        B d[NL], u[NL], v[NL];
        double dx, dy;
    };
    auto load = [&](int r, unsigned b, Row &R) {   // b: an opaque zero
        const unsigned e = row(r) + b, eu = row(r - 1) + b, ev = row(r - 2) + b;
#pragma unroll
        for (int q = 0; q < NI; q++) {
            R.p[q] = el(A.pfull + oi[q], e * 8);
            R.z[q] = el(A.phi + oi[q], e * 8);
        }
#pragma unroll
        for (int q = 0; q < NL; q++) {
            R.d[q] = el(A.delp + ol[q], e * (unsigned)sizeof(B));
            R.u[q] = el(A.u + ol[q], eu * (unsigned)sizeof(B));
            R.v[q] = el(A.v + ol[q], ev * (unsigned)sizeof(B));
        }
        R.dx = el(M.m[M_DX] + o2, eu * 8);
        R.dy = el(M.m[M_DY] + o2, ev * 8);
        if (G.cube && (r < 0 || r >= n)) {
            const int rr = min(max(r, -3), n + 2);
            if (in_corner(G, SC, ic, rr)) {
#pragma unroll
                for (int q = 0; q < NI; q++) {
                    R.p[q] = sv(G, A.pfull + oi[q] + hb, SC, ic, rr, 0);
                    R.z[q] = sv(G, A.phi + oi[q] + hb, SC, ic, rr, 0);
                }
#pragma unroll
                for (int q = 0; q < NL; q++) R.d[q] = sv(G, A.delp + ol[q] + hb, SC, ic, rr, 0);
            }
        }
    };
    // mean of the three cells around a cube vertex
    auto vertex = [&](auto *pl, int m) -> double {
        const int ci[4] = {i - 1, i, i, i - 1}, cj[4] = {m - 1, m - 1, m, m};
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < 4; q++)
            if (!in_corner(G, SC, ci[q], cj[q])) sum += (double)AT(pl, ci[q], cj[q]);
        return fdiv(sum, 3.0);
    };

    double x1[NF], x2[NF], x3[NF], cp[NF];   // x passes of rows r - 1, r - 2, r - 3; corners of row r - 2
#pragma unroll
    for (int f = 0; f < NF; f++) x1[f] = x2[f] = x3[f] = cp[f] = 0.0;
    Row cur, nxt;
    unsigned zero = 0;
    load(j0 - 2, zero, cur);
    const int rend = min(j1, n) + 2;   // rows j0 - 2 .. ; corners j0 .. min(j1, n)
    for (int r = j0 - 2; r < rend; r++) {
        __asm__ volatile("" : "+v"(zero));   // addresses are formed per row, not carried in registers
        if (r + 1 < rend) load(r + 1, zero, nxt);
        const bool rin = r >= 0 && r < n;
        const int m = r - 1;
        double x0[NF], c[NF];
#pragma unroll
        for (int f = 0; f < NF; f++) {
            const double a = f < NI ? cur.p[f] : f < 2 * NI ? cur.z[f - NI] : (double)cur.d[f - 2 * NI];
            const double aw = west(a), aww = west(aw), ae = east(a);
            x0[f] = face_mean<EI>(aww, aw, a, ae, i, n, rin);
            c[f] = face_mean<EI>(x3[f], x2[f], x1[f], x0[f], m, n, true);
        }
        if (G.cube && (m == 0 || m == n) && m >= j0 && (i == 0 || i == n)) {
#pragma unroll
            for (int q = 0; q < NI; q++) {
                c[q] = vertex(A.pfull + oi[q] + hb, m);
                c[NI + q] = vertex(A.phi + oi[q] + hb, m);
            }
#pragma unroll
            for (int q = 0; q < NL; q++) c[2 * NI + q] = vertex(A.delp + ol[q] + hb, m);
        }
        double ce[NF];
#pragma unroll
        for (int f = 0; f < NF; f++) ce[f] = east(c[f]);
#pragma unroll
        for (int q = 0; q < NL; q++) {
            if (k + q >= nz) continue;
            const int d = 2 * NI + q, z = NI + q;
            if (fu && m >= j0 && m < j1)
                el(A.u + ol[q], row(m) * (unsigned)sizeof(B)) =
                    cur.u[q] + (B)layer_pgf(A.bdt, cur.dx, c[d], ce[d], c[z], c[z + 1], ce[z], ce[z + 1], c[q], c[q + 1],
                                            ce[q], ce[q + 1]);
            if (mine && m > j0)
                el(A.v + ol[q], row(m - 1) * (unsigned)sizeof(B)) =
                    cur.v[q] + (B)layer_pgf(A.bdt, cur.dy, cp[d], c[d], cp[z], cp[z + 1], c[z], c[z + 1], cp[q],
                                            cp[q + 1], c[q], c[q + 1]);
        }
#pragma unroll
        for (int f = 0; f < NF; f++) {
            x3[f] = x2[f];
            x2[f] = x1[f];
            x1[f] = x0[f];
            cp[f] = c[f];
        }
        cur = nxt;
    }
}

template <class B, bool EI>
DEVI void k_nhpgrad(Bk bk, Geo G, MetD M, NhArgs<B> A)
{
    if (A.layers == 2) nhpgrad_body<B, EI, 2>(bk, G, M, A);
    else nhpgrad_body<B, EI, 1>(bk, G, M, A);
}

template <class B>
void nh_grad(const fv3_grid *g, const NhArgs<B> &args, hipStream_t st)
{
    NhArgs<B> a = args;
    MetD M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = g->met[m];
    const int pts = g->n + 1;
    // two layers a wavefront where one segment of rows each still gives three
    // quarters of a wavefront per SIMD (one / two layers, us: C192 x 79 233 / 203,
    // C96 x 79 FP64 82 / 78, C48 x 79 24.5 / 26.4, periodic 48 x 8 5.8 / 7.5)
    a.layers = (long)g->T * g->nz * ((pts + 57) / 58) >= 768 ? 2 : 1;
    const int nzb = (g->nz + 4 * a.layers - 1) / (4 * a.layers);
    // wavefronts per round for the split, by measurement: the kernel, which holds
    // both bodies, fits three, but told so it takes C192 x 79 mixed from 205 to
    // 222 us and FP64 from 269 to 284 (C140 x 79 from 143 to 120 and from 202 to
    // 177; within 2% elsewhere between 48 x 8 and C384 x 20)
    march_shape(pts, (long)g->T * nzb * 4, 4, a.layers == 2 ? 2 : 4, a.strips, a.width, a.segs, a.rows);
    const dim3 grd((unsigned)((long)a.strips * a.segs * g->T * nzb)), blk(256);
    if (g->p.edge_interp && g->p.kind == FV3_GRID_CUBED_SPHERE)
        launch_fn<k_nhpgrad<B, true>>("k_nhpgrad", grd, blk, st, g->geo, M, a);
    else
        launch_fn<k_nhpgrad<B, false>>("k_nhpgrad", grd, blk, st, g->geo, M, a);
}
template void nh_grad<float>(const fv3_grid *, const NhArgs<float> &, hipStream_t);
template void nh_grad<double>(const fv3_grid *, const NhArgs<double> &, hipStream_t);

}  // namespace fv3
