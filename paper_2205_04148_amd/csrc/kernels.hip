// HIP kernels of the FV3 acoustic substep loop and tracer transport (gfx950).
//
// Data layout: every field is [tile][level][row][column], column index i
// contiguous (coalesced across the 64 lanes of a wavefront), halo of 3 points,
// rows padded to 128 bytes with interior i = 0 aligned.  Kernels are
// templated on the bulk type B (double, or float for the mixed-precision
// build); the column solves, vertical scans, pressure gradients and mass-flux
// accumulators are always FP64.
//
// Stencil kernels of this file work on one (tile, level) plane per grid z index.
// c_sw, the flux-form transports, nh_p_grad and the column solves have files of
// their own (csw, transport, nhgrad, column); with one-sided faces at tile edges
// (edge_ppm) the transport fv_tp_2d (paper Sec. IX-C) is the kernel here: a cell
// tile with its 3-point halo is staged in LDS, and the outer fluxes, inner
// advective updates, final fluxes and the flux-divergence update of the
// transported field all run out of LDS.  Corner blocks of cube tiles
// are never stored: reads of them are remapped to the adjacent edge halo
// rotated about the cube vertex, in the x-sweep or y-sweep sense of the
// reading stencil (generalising the corner statement of Sec. VII-C).
//
// The order of the stages inside a substep follows the FV3 acoustic loop
// (Sec. II): halo A, c_sw, dz_c + riem_solver_c, p_grad_c, halo B, d_sw,
// dz_d + riem_solver3, halo C, nh_p_grad.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <utility>
#include <string>
#include <vector>

#include "fv3_internal.hpp"
#include "column.hpp"
#include "csw.hpp"
#include "nhgrad.hpp"
#include "launch.hpp"
#include "transport.hpp"

namespace fv3 {

// ---------------------------------------------------------- launch timing
static struct {
    bool on = false;
    std::string filter;
    std::vector<TimingRec> recs;
} g_timing;

bool timing_wanted(const char *name)
{
    return g_timing.on && std::strstr(name, g_timing.filter.c_str()) != nullptr;
}
void timing_begin(const char *name, hipStream_t st, TimingRec &r)
{
    r.name = name;
    (void)hipEventCreate(&r.a);
    (void)hipEventCreate(&r.b);
    (void)hipEventRecord(r.a, st);
}
void timing_end(hipStream_t st, TimingRec &r)
{
    (void)hipEventRecord(r.b, st);
    g_timing.recs.push_back(r);
}

thread_local Recorder *g_rec = nullptr;

// marks the boundaries entry | substep | exit of the recorded sequence
static void rec_mark()
{
    if (!g_rec) return;
    Recorder &R = *g_rec;
    if (R.member == 0) R.marks.push_back(R.pos);
    else if (R.mark >= R.marks.size() || R.marks[R.mark] != R.pos) R.bad = true;
    R.mark++;
}

// plain __global__ kernels outside the substep path (reductions)
template <class Kern, class... A>
static void launch2d_native(const char *name, Kern kern, int ilo, int ihi, int jlo, int jhi, int planes,
                            hipStream_t st, A... a)
{
    dim3 blk(64, 4, 1);
    dim3 grd((unsigned)((ihi - ilo + 64) / 64), (unsigned)((jhi - jlo + 4) / 4), (unsigned)planes);
    bool tm = timing_wanted(name);
    TimingRec r;
    if (tm) timing_begin(name, st, r);
    hipLaunchKernelGGL(kern, grd, blk, 0, st, ilo, ihi, jlo, jhi, a...);
    if (tm) timing_end(st, r);
}

// ====================================================================
// 1-D PPM face value: face between cells m-1 and m along a sweep, cell
// values q0..q5 = cells m-3..m+2, Courant number c, order ORD.
//  8 monotone: limited slope per cell (zero at extrema), fourth-order edge
//    values, edge deviations clipped to twice the slope with the slope's
//    sign, mean of the parabola over the swept part of the upwind cell;
//  6 unlimited: slopes (q+ - q-)/4 and the edge deviations as they come;
//  5 2dx-filtered: order 6, but the upwind cell mean where that cell and a
//    neighbour are both strict local extrema (an oscillation over 2 cells);
//  7 positive-definite (tracers): order 6 with the parabola of a cell of
//    non-negative mean q scaled about q by q / (q - min) where its minimum
//    over the cell is negative (Zhang & Shu's scaling limiter).
// ====================================================================
template <class T>
DEVI T lslope(T a, T b, T c)
{
    // zero at an extremum of (a, b, c): then min(mx - b, b - mn) is zero
    T d = (c - a) * (T)0.25;
    T mx = fmax(a, fmax(b, c)), mn = fmin(a, fmin(b, c));
    return copysign(fmin(fabs(d), fmin(mx - b, b - mn)), d);
}

// Face value from the upwind cell q's parabola (neighbours a, b | d, e), with
// c the signed Courant number.  For the downwind orientation the parabola's
// edge deviations swap roles and the swept fraction is |c|:
// q + (1 - |c|) (e - |c| (bl + br)), e = br for c > 0 and bl otherwise.
template <int ORD, class T>
DEVI T ppm_up(T a, T b, T q, T d, T e, T c)
{
    const T third = (T)1 / (T)3;
    if constexpr (ORD == 5) {
        const bool xb = (b - a) * (q - b) < (T)0, xq = (q - b) * (d - q) < (T)0, xd = (d - q) * (e - d) < (T)0;
        if (xq && (xb || xd)) return q;
    }
    T bl, br;
    if constexpr (ORD == 8) {
        const T dl = lslope(a, b, q), dm = lslope(b, q, d), dr = lslope(q, d, e);
        const T al = (T)0.5 * (b + q) + (dl - dm) * third;
        const T ar = (T)0.5 * (q + d) + (dm - dr) * third;
        // deviations clipped to twice the slope, with the slope's sign (zero slope: zero)
        const T a2 = (T)2 * fabs(dm);
        bl = copysign(fmin(a2, fabs(al - q)), -dm);
        br = copysign(fmin(a2, fabs(ar - q)), dm);
    } else {
        const T qt = (T)0.25;
        const T dl = (q - a) * qt, dm = (d - b) * qt, dr = (e - q) * qt;
        bl = (T)0.5 * (b + q) + (dl - dm) * third - q;
        br = (T)0.5 * (q + d) + (dm - dr) * third - q;
    }
    if constexpr (ORD == 7) {
        if (q >= (T)0) {
            // minimum over the cell: an edge, or the vertex when it is a
            // minimum (a6 < 0) inside the cell (|aR - aL| < -a6)
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
    const T cc = fabs(c);
    return q + ((T)1 - cc) * ((c > 0 ? br : bl) - cc * (bl + br));
}

template <int ORD, class T>
DEVI T ppm6(T q0, T q1, T q2, T q3, T q4, T q5, T c)
{
    // Branch-free: select the upwind cell's five-point neighbourhood (cell
    // m-1 for c > 0, else cell m), then one evaluation.
    const bool pos = c > 0;
    return ppm_up<ORD>(pos ? q0 : q1, pos ? q1 : q2, pos ? q2 : q3, pos ? q3 : q4, pos ? q4 : q5, c);
}

// The same from six cells m-3..m+2 stored S apart from p (in LDS): the upwind
// neighbourhood is selected by its address, five loads instead of six.
template <int S, int ORD, class T>
DEVI T ppm_lds(const T *p, T c)
{
    const T *u = p + (c > 0 ? 0 : S);
    return ppm_up<ORD>(u[0], u[S], u[2 * S], u[3 * S], u[4 * S], c);
}

// Face value next to a cube tile edge (option edge_ppm, Putman & Lin 2007).
// p holds the six cells m-3..m+2 of the sweep, S apart; w their widths along
// the sweep, ws apart.  Window interface pe (between window cells pe-1 and
// pe, 1 <= pe <= 5) is the edge; the tile lies at cells >= pe (west) or
// below pe.  The edge values of the three interfaces around the edge are
// one-sided: at the edge, the mean of the linear extrapolations from the two
// cells on either side (by distance); next to it, three cells of its own
// side, (3 q_near + 11 q_far) / 14 -+ (4/7) times the far cell's slope.
// Order 8 leaves the deviations of the two cells beside the edge and of the
// second cell inside the tile unclipped and makes their parabolas monotone
// (Colella & Woodward 1984).  Written without dynamically indexed arrays.
template <int ORD, class T>
DEVI T ppm_edge(const T *p, int S, const T *w, int ws, T c, int pe, bool west)
{
    T q[6], x[6], dm[6], al[6];
#pragma unroll
    for (int k = 0; k < 6; k++) {
        q[k] = p[k * S];
        x[k] = w[k * ws];
    }
    const bool pos = c > 0;
    if constexpr (ORD == 5) {
        const bool x1 = (q[1] - q[0]) * (q[2] - q[1]) < (T)0, x2 = (q[2] - q[1]) * (q[3] - q[2]) < (T)0;
        const bool x3 = (q[3] - q[2]) * (q[4] - q[3]) < (T)0, x4 = (q[4] - q[3]) * (q[5] - q[4]) < (T)0;
        if (pos ? (x2 && (x1 || x3)) : (x3 && (x2 || x4))) return pos ? q[2] : q[3];
    }
#pragma unroll
    for (int k = 1; k <= 4; k++)
        dm[k] = ORD == 8 ? lslope(q[k - 1], q[k], q[k + 1]) : (q[k + 1] - q[k - 1]) * (T)0.25;
    const T third = (T)1 / (T)3, r14 = (T)1 / (T)14, f47 = (T)4 / (T)7;
#pragma unroll
    for (int k = 2; k <= 4; k++) {
        T v = (T)0.5 * (q[k - 1] + q[k]) + (dm[k - 1] - dm[k]) * third;
        if (k == pe) {
            const T lo = (((T)2 * x[k - 1] + x[k - 2]) * q[k - 1] - x[k - 1] * q[k - 2]) / (x[k - 2] + x[k - 1]);
            const T hi = (((T)2 * x[k] + x[k + 1]) * q[k] - x[k] * q[k + 1]) / (x[k] + x[k + 1]);
            v = (T)0.5 * (lo + hi);
        } else if (k == pe - 1) {
            v = ((T)3 * q[k] + (T)11 * q[k - 1]) * r14 + f47 * dm[k - 1];
        } else if (k == pe + 1) {
            v = ((T)3 * q[k - 1] + (T)11 * q[k]) * r14 - f47 * dm[k];
        }
        al[k] = v;
    }
    const int s = pos ? 2 : 3;
    const T qs = pos ? q[2] : q[3], ds = pos ? dm[2] : dm[3];
    const T aL = pos ? al[2] : al[3], aR = pos ? al[3] : al[4];
    const bool edge_cell = s == pe - 1 || s == pe || s == (west ? pe + 1 : pe - 2);
    T bl = aL - qs, br = aR - qs;
    if constexpr (ORD == 8) {
        if (!edge_cell) {
            const T a2 = (T)2 * fabs(ds);
            bl = copysign(fmin(a2, fabs(bl)), -ds);
            br = copysign(fmin(a2, fabs(br)), ds);
        } else if (bl * br >= (T)0) {
            bl = br = (T)0;
        } else {
            const T da = br - bl, a6 = (T)-3 * (bl + br);
            if (a6 * da > da * da) bl = (T)-2 * br;
            else if (a6 * da < -(da * da)) br = (T)-2 * bl;
        }
    }
    if constexpr (ORD == 7) {
        if (qs >= (T)0) {
            const T eL = qs + bl, eR = qs + br, a6 = (T)-3 * (bl + br), da = eR - eL;
            T mn = fmin(eL, eR);
            if (a6 < (T)0 && fabs(da) < -a6) mn = fmin(mn, qs + da * da / ((T)4 * a6) + a6 / (T)12);
            if (mn < (T)0) {
                const T th = qs / (qs - mn);
                bl *= th;
                br *= th;
            }
        }
    }
    const T cc = fabs(c);
    return qs + ((T)1 - cc) * ((pos ? br : bl) - cc * (bl + br));
}

// Window position of a tile edge for face m of a sweep over n cells, or 0
// when the face has no edge cell upwind (faces 0, 1, 2 and n-2, n-1, n do).
DEVI int edge_pe(int m, int n, bool &west)
{
    west = m <= 2;
    if (m >= 0 && m <= 2) return 3 - m;
    if (m >= n - 2 && m <= n) return n - m + 3;
    return 0;
}
DEVI bool edge_face(int m, int n) { return m <= 2 || m >= n - 2; }
// the k-th (0..5) face with an edge cell upwind: 0, 1, 2, n-2, n-1, n
DEVI int edge_face_at(int k, int n) { return k < 3 ? k : n - 5 + k; }

// ====================================================================
// Halo exchange: plan-driven copies from the neighbour tile's interior
// (orientation transform folded into the plan for vector pairs).
// ====================================================================
template <class T>
DEVI void k_halo_scalar(Bk bk, Geo G, const HaloEnt *__restrict__ plan, int count, T *f, int L)
{
    int e = bk.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    int k = bk.y;
    HaloEnt h = plan[e];
    f[pidx(G, L, h.dt, k) + h.di] = f[pidx(G, L, h.st, k) + h.si];
}

template <class T>
DEVI void k_halo_pair(Bk bk, Geo G, const HaloEnt *__restrict__ plan, int count, T *fx, T *fy, int L)
{
    int e = bk.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    int k = bk.y;
    HaloEnt h = plan[e];
    const T *src = (h.sel & 1) ? fy : fx;
    T *dst = (h.sel & 4) ? fy : fx;
    T v = src[pidx(G, L, h.st, k) + h.si];
    dst[pidx(G, L, h.dt, k) + h.di] = (h.sel & 2) ? -v : v;
}

// up to four fields of one type and level count in one launch: grid y runs
// over (field, level)
template <class T>
struct FieldSet {
    T *p[4];
};
template <class T>
DEVI void k_halo_set(Bk bk, Geo G, const HaloEnt *__restrict__ plan, int count, FieldSet<T> F, int L)
{
    int e = bk.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    int q = (int)bk.y / L, k = (int)bk.y % L;
    T *f = q == 0 ? F.p[0] : q == 1 ? F.p[1] : q == 2 ? F.p[2] : F.p[3];
    HaloEnt h = plan[e];
    f[pidx(G, L, h.dt, k) + h.di] = f[pidx(G, L, h.st, k) + h.si];
}
template <class T>
static void halo_set(const fv3_grid *g, FieldSet<T> F, int nf, int L, hipStream_t st)
{
    if (g->planC.count == 0) return;
    launch_fn<k_halo_set<T>>("k_halo_scalar", dim3((g->planC.count + 255) / 256, L * nf), dim3(256), st,
                 g->geo, (const HaloEnt *)g->planC.d, g->planC.count, F, L);
}

template <class T>
static void halo_scalar(const fv3_grid *g, T *f, int L, hipStream_t st)
{
    if (g->planC.count == 0) return;
    launch_fn<k_halo_scalar<T>>("k_halo_scalar", dim3((g->planC.count + 255) / 256, L), dim3(256), st,
                 g->geo, (const HaloEnt *)g->planC.d, g->planC.count, f, L);
}
// corner (B-grid) scalar field
template <class T>
static void halo_corner(const fv3_grid *g, T *f, int L, hipStream_t st)
{
    if (g->planB.count == 0) return;
    launch_fn<k_halo_scalar<T>>("k_halo_corner", dim3((g->planB.count + 255) / 256, L), dim3(256), st,
                 g->geo, (const HaloEnt *)g->planB.d, g->planB.count, f, L);
}
template <class T>
static void halo_pair(const fv3_grid *g, const Plan &p, T *fx, T *fy, int L, hipStream_t st)
{
    if (p.count == 0) return;
    launch_fn<k_halo_pair<T>>("k_halo_pair", dim3((p.count + 255) / 256, L), dim3(256), st, g->geo,
                 (const HaloEnt *)p.d, p.count, fx, fy, L);
}

// ====================================================================
// Pressure gradients
// ====================================================================
// Finite-volume pressure gradient between two columns W, E over one layer:
// contour integral of p dPhi around the quadrilateral of the two columns'
// interfaces k, k+1, over the mean layer mass and the distance L.
DEVI double pgf(double dt, double L, double dW, double dE, double zW0, double zW1, double zE0,
                double zE1, double pW0, double pW1, double pE0, double pE1)
{
    return dt / (L * (dW + dE)) * ((zW1 - zE0) * (pE1 - pW0) + (zW0 - zE1) * (pW1 - pE0));
}

// p_grad_c on the interior C-grid faces with the half-step cells' pressure
// and geopotential; layer mass weights from delpc.  Each thread walks PGK
// consecutive layers of its point: the interface below one layer is the
// interface above the next, so its pressure and geopotential are carried
// instead of loaded again (the face metric too).
#ifndef FV3_PGK
#define FV3_PGK 4
#endif
constexpr int PGK = FV3_PGK;
template <class B>
DEVI void k_pgradc(KARGS, Geo G, MetD M, double dt2, const B *delpc, const double *pkc,
                         const double *gz, B *uc, B *vc)
{
    const int i = ib + (int)(bk.x * blockDim.x + threadIdx.x);
    const int j = jlo + (int)(bk.y * blockDim.y + threadIdx.y);
    if (i < ilo || i > ihi || j > jhi) return;
    const int n = G.n, nz = G.nz, nzb = (nz + PGK - 1) / PGK;
    const int t = (int)bk.z / nzb, k0 = ((int)bk.z % nzb) * PGK;
    const bool fx = j < n, fy = i < n;   // x-face (i, j) and y-face (i, j) of this point
    if (!fx && !fy) return;
    const double dxc = fx ? AT(MP(M, M_DXC), i, j) : 0.0, dyc = fy ? AT(MP(M, M_DYC), i, j) : 0.0;
    // cells W = (i - 1, j), C = (i, j), S = (i, j - 1) at the interface above the layer
    long oi = pidx(G, nz + 1, t, k0);
    double zW = 0, pW = 0, zS = 0, pS = 0;
    if (fx) { zW = AT(gz + oi, i - 1, j); pW = AT(pkc + oi, i - 1, j); }
    if (fy) { zS = AT(gz + oi, i, j - 1); pS = AT(pkc + oi, i, j - 1); }
    double zC = AT(gz + oi, i, j), pC = AT(pkc + oi, i, j);
    const int k1 = k0 + PGK < nz ? k0 + PGK : nz;
    for (int k = k0; k < k1; k++) {
        const long o = pidx(G, nz, t, k), o1 = pidx(G, nz + 1, t, k + 1);
        const B *D = delpc + o;
        double zW1 = 0, pW1 = 0, zS1 = 0, pS1 = 0;
        if (fx) { zW1 = AT(gz + o1, i - 1, j); pW1 = AT(pkc + o1, i - 1, j); }
        if (fy) { zS1 = AT(gz + o1, i, j - 1); pS1 = AT(pkc + o1, i, j - 1); }
        const double zC1 = AT(gz + o1, i, j), pC1 = AT(pkc + o1, i, j);
        const double dC = (double)AT(D, i, j);
        if (fx)
            AT(uc + o, i, j) += (B)pgf(dt2, dxc, (double)AT(D, i - 1, j), dC, zW, zW1, zC, zC1, pW, pW1, pC, pC1);
        if (fy)
            AT(vc + o, i, j) += (B)pgf(dt2, dyc, (double)AT(D, i, j - 1), dC, zS, zS1, zC, zC1, pS, pS1, pC, pC1);
        zW = zW1; pW = pW1; zS = zS1; pS = pS1; zC = zC1; pC = pC1;
    }
}

// ====================================================================
// fv_tp_2d (Sec. IX-C) with one-sided faces at cube tile edges (edge_ppm):
// Lin-Rood flux-form transport on one level, fused.  A cell tile (32 x 16 in FP32, 32 x 8 in FP64) plus 3-point halo is staged
// in LDS in both sweep views; outer PPM fluxes, inner advective half updates, final averaged and
// weighted fluxes, then an epilogue that applies the flux divergence:
//   EPI_FLUX   write the fluxes only
//   EPI_DELP   write fluxes, accumulate them (mass fluxes, Courant numbers),
//              new delp = delp + div F / area
//   EPI_MASSW  mass-weighted update (q delp_old area + div F) / (delp_new area)
//   EPI_ADV    advective update (q area + div F) / (area + div of area fluxes)
//   EPI_TRACER (q dp1 area + div F) / (dp2 area)
// With `iface`, the Courant numbers and area fluxes of plane k are the mean
// of layers k-1 and k (plane 0: layer 0), for interface heights.
// ====================================================================
enum { EPI_FLUX = 0, EPI_DELP = 1, EPI_MASSW = 2, EPI_ADV = 3, EPI_TRACER = 4 };
// Cell tile per field precision (measured on MI355X at C192 x 79: the FP64
// tile is smaller so that four blocks fit a CU's LDS at 256 threads each).
constexpr int FNT = 256;
template <class T>
struct FvTile {
    static constexpr int X = 32, Y = 16;
};
template <>
struct FvTile<double> {
    static constexpr int X = 32, Y = 8;
};

template <class T, class C, class M>
struct FvArgs {
    const T *q;
    int Lq;
    const C *crx, *cry, *xfx, *yfx;
    int Lc, iface;
    const M *mx, *my;      // optional flux weights (mass fluxes)
    const T *area;         // area metric (type T)
    const T *dxa, *dya;    // cell widths along x and y (type T; tile-edge PPM)
    int epi;
    T *FX, *FY;            // flux outputs (may be null)
    int edges_only;        // write the flux outputs on tile-edge faces only
    T *qout;               // cell output, Lq levels
    const T *dold, *dnew;  // EPI_MASSW
    const double *dp1, *dp2;            // EPI_TRACER
    double *mfx, *mfy;     // EPI_DELP accumulators
    C *cxa, *cya;
};

// Loads and stores through a block-uniform base pointer and a 32-bit
// unsigned element offset (one VALU add per access instead of 64-bit
// address arithmetic).
template <class T>
DEVI T ldo(const T *base, unsigned e)
{
    return *(const T *)((const char *)base + e * (unsigned)sizeof(T));
}
template <class T>
DEVI void sto(T *base, unsigned e, T v)
{
    *(T *)((char *)base + e * (unsigned)sizeof(T)) = v;
}

template <class T, class C>
DEVI T ccr(const C *a, const C *a0, unsigned idx, int avg)
{
    if (avg) return (T)(0.5 * ((double)ldo(a0, idx) + (double)ldo(a, idx)));
    return (T)ldo(a, idx);
}

// The transport tile in LDS (one instance per block, shared by both
// instantiations of the body).
template <class T>
struct FvLds {
    static constexpr int FTX = FvTile<T>::X, FTY = FvTile<T>::Y;
    static constexpr int QW = FTX + 6, QH = FTY + 6;
    static constexpr int YW = FTX + 6, YH = FTY + 1;   // y-faces: cols i0-3..i0+FTX+2, rows j0..j0+FTY
    static constexpr int XW = FTX + 1, XH = FTY + 6;   // x-faces: cols i0..i0+FTX, rows j0-3..j0+FTY+2
    T sQ[QH * QW], sQy[QH * QW], sAR[QH * QW];
    T sCY[YH * YW], sYF[YH * YW], sFy[YH * YW];
    T sCX[XH * XW], sXF[XH * XW], sFx[XH * XW];
    T sQi[FTY * QW];                // cells: cols i0-3..i0+FTX+2, rows j0..j0+FTY-1
    T sQj[QH * FTX];                // cells: cols i0..i0+FTX-1, rows j0-3..j0+FTY+2
};

// CORNER: the block's staging window reaches a cube corner block (only
// blocks at the four corners of a tile), so its field reads go through the
// corner views; every other block reads the plane directly.
template <class T, class C, class M, int EPI, int ORD, bool CORNER>
DEVI void fvtp_body(Bk bk, const Geo &G, const FvArgs<T, C, M> &A, FvLds<T> &L)
{
    constexpr int FTX = FvTile<T>::X, FTY = FvTile<T>::Y;
    constexpr int QW = FvLds<T>::QW, QH = FvLds<T>::QH;
    constexpr int YW = FvLds<T>::YW, YH = FvLds<T>::YH;
    constexpr int XW = FvLds<T>::XW, XH = FvLds<T>::XH;
    constexpr int N4X = (FTY * XW + FNT - 1) / FNT, N4Y = (YH * FTX + FNT - 1) / FNT;
    constexpr int N5 = (FTY * FTX + FNT - 1) / FNT;
    T *sQ = L.sQ, *sQy = L.sQy, *sAR = L.sAR, *sCY = L.sCY, *sYF = L.sYF, *sFy = L.sFy;
    T *sCX = L.sCX, *sXF = L.sXF, *sFx = L.sFx, *sQi = L.sQi, *sQj = L.sQj;
    const int n = G.n, tid = threadIdx.x;
    const int i0 = bk.x * FTX, j0 = bk.y * FTY;
    const int t = bk.z / A.Lc, k = bk.z % A.Lc;
    // plane pointers (block-uniform); the staged ones are rebased to the
    // halo corner (-3, -3) so that every offset is a non-negative 32-bit value
    const int P = (int)G.pitch;
    const unsigned hb = 3u * (unsigned)P + 3u;   // rebase of the staging windows
    const T *Q = A.q + pidx(G, A.Lq, t, k);
    const long oc = pidx(G, A.Lc, t, k);
    const int avg = EPI == EPI_ADV && A.iface && k > 0;   // set only for the interface heights
    const long ob = avg ? pidx(G, A.Lc, t, k - 1) : oc;
    const T *AR = A.area + G.off0 + (long)t * G.lev;
    const T *DXA = A.dxa + G.off0 + (long)t * G.lev;
    const T *DYA = A.dya + G.off0 + (long)t * G.lev;
    const T *Qh = Q - hb, *ARh = AR - hb;
    const C *cryh = A.cry + oc - hb, *yfxh = A.yfx + oc - hb, *crxh = A.crx + oc - hb, *xfxh = A.xfx + oc - hb;
    const C *cry0h = A.cry + ob - hb, *yfx0h = A.yfx + ob - hb, *crx0h = A.crx + ob - hb, *xfx0h = A.xfx + ob - hb;
    const M *MX = A.mx ? A.mx + oc : nullptr, *MY = A.my ? A.my + oc : nullptr;
    using PT = typename std::conditional<EPI == EPI_TRACER, double, T>::type;

    // 0. per-thread prefetch of the global operands of phases 4 and 5, in
    //    their storage types (with the delp epilogue also the old values of
    //    the flux accumulators that phase 4 adds to: their loads would
    //    otherwise wait behind the previous face's stores)
    M wx[N4X], wy[N4Y];
    constexpr int NAX = EPI == EPI_DELP ? N4X : 1, NAY = EPI == EPI_DELP ? N4Y : 1;
    double amx[NAX], amy[NAY];
    C acx[NAX], acy[NAY];
    PT pa[N5], pb[N5];
#pragma unroll
    for (int m = 0; m < N4X; m++) {
        int e = tid + m * FNT, r = e / XW, c = e - r * XW;
        int i = i0 + c, j = j0 + r;
        const bool in = e < FTY * XW && i <= n && j < n;
        wx[m] = (MX && in) ? ldo(MX, (unsigned)(j * P + i)) : (M)0;
        if constexpr (EPI == EPI_DELP) {
            // the faces phase 4 writes: c < FTX, or the last face i == n
            const bool own = in && (c < FTX || i == n) && !edge_face(i, n);
            amx[m] = own ? ldo(A.mfx + oc, (unsigned)(j * P + i)) : 0.0;
            acx[m] = own ? ldo(A.cxa + oc, (unsigned)(j * P + i)) : (C)0;
        }
    }
#pragma unroll
    for (int m = 0; m < N4Y; m++) {
        int e = tid + m * FNT, r = e / FTX, c = e - r * FTX;
        int i = i0 + c, j = j0 + r;
        const bool in = e < YH * FTX && i < n && j <= n;
        wy[m] = (MY && in) ? ldo(MY, (unsigned)(j * P + i)) : (M)0;
        if constexpr (EPI == EPI_DELP) {
            const bool own = in && (r < FTY || j == n) && !edge_face(j, n);
            amy[m] = own ? ldo(A.mfy + oc, (unsigned)(j * P + i)) : 0.0;
            acy[m] = own ? ldo(A.cya + oc, (unsigned)(j * P + i)) : (C)0;
        }
    }
#pragma unroll
    for (int m = 0; m < N5; m++) {
        int e = tid + m * FNT, r = e / FTX, c = e - r * FTX;
        int i = i0 + c, j = j0 + r;
        bool in = e < FTY * FTX && i < n && j < n;
        unsigned ci = (unsigned)(j * P + i);
        pa[m] = (PT)0;
        pb[m] = (PT)0;
        if constexpr (EPI == EPI_MASSW) {
            if (in) {
                pa[m] = ldo(A.dold + oc, ci);
                pb[m] = ldo(A.dnew + oc, ci);
            }
        } else if constexpr (EPI == EPI_TRACER) {
            if (in) {
                pa[m] = ldo(A.dp1 + oc, ci);
                pb[m] = ldo(A.dp2 + oc, ci);
            }
        }
    }
    // 1. stage the field (both sweep views), the area, the Courant numbers and
    //    the area fluxes of the tile and its halo: every load of the thread
    //    is issued before the first LDS write, so that they are all in flight
    //    together
    {
        constexpr int NSQ = (QH * QW + FNT - 1) / FNT, NSY = (YH * YW + FNT - 1) / FNT;
        constexpr int NSX = (XH * XW + FNT - 1) / FNT;
        T qx[NSQ], qy[NSQ], qa[NSQ], cy[NSY], fy[NSY], cx[NSX], fx[NSX];
#pragma unroll
        for (int m = 0; m < NSQ; m++) {
            const int e = tid + m * FNT, r = e / QW, c = e - r * QW;
            const int i = i0 - 3 + c, j = j0 - 3 + r;
            T vx = 0, vy = 0, ar = 0;
            if (e < QH * QW && i <= n + 2 && j <= n + 2) {
                if (CORNER && in_corner(G, SC, i, j)) {
                    vx = sv(G, Q, SC, i, j, 0);
                    vy = sv(G, Q, SC, i, j, 1);
                } else {
                    const unsigned u = (unsigned)((j + 3) * P + (i + 3));
                    vx = vy = ldo(Qh, u);
                    ar = ldo(ARh, u);
                }
            }
            qx[m] = vx;
            qy[m] = vy;
            qa[m] = ar;
        }
#pragma unroll
        for (int m = 0; m < NSY; m++) {
            const int e = tid + m * FNT, r = e / YW, c = e - r * YW;
            const int i = i0 - 3 + c, j = j0 + r;
            T cr = 0, fl = 0;
            if (e < YH * YW && i <= n + 2 && j <= n) {
                const unsigned u = (unsigned)((j + 3) * P + (i + 3));
                cr = ccr<T>(cryh, cry0h, u, avg);
                fl = ccr<T>(yfxh, yfx0h, u, avg);
            }
            cy[m] = cr;
            fy[m] = fl;
        }
#pragma unroll
        for (int m = 0; m < NSX; m++) {
            const int e = tid + m * FNT, r = e / XW, c = e - r * XW;
            const int i = i0 + c, j = j0 - 3 + r;
            T cr = 0, fl = 0;
            if (e < XH * XW && i <= n && j <= n + 2) {
                const unsigned u = (unsigned)((j + 3) * P + (i + 3));
                cr = ccr<T>(crxh, crx0h, u, avg);
                fl = ccr<T>(xfxh, xfx0h, u, avg);
            }
            cx[m] = cr;
            fx[m] = fl;
        }
#pragma unroll
        for (int m = 0; m < NSQ; m++) {
            const int e = tid + m * FNT;
            if (e < QH * QW) {
                sQ[e] = qx[m];
                sQy[e] = qy[m];
                sAR[e] = qa[m];
            }
        }
#pragma unroll
        for (int m = 0; m < NSY; m++) {
            const int e = tid + m * FNT;
            if (e < YH * YW) {
                sCY[e] = cy[m];
                sYF[e] = fy[m];
            }
        }
#pragma unroll
        for (int m = 0; m < NSX; m++) {
            const int e = tid + m * FNT;
            if (e < XH * XW) {
                sCX[e] = cx[m];
                sXF[e] = fx[m];
            }
        }
    }
    __syncthreads();
    // 2. outer fluxes of the field (unrolled: the LDS reads of the next
    //    faces overlap the arithmetic of the current one)
#pragma unroll
    for (int m = 0; m < (YH * YW + FNT - 1) / FNT; m++) {
        const int e = tid + m * FNT;
        if (e >= YH * YW) break;
        int r = e / YW, c = e - r * YW;
        int i = i0 - 3 + c, j = j0 + r;
        T f = 0;
        if (i <= n + 2 && j <= n) {
            const T *col = sQy + r * QW + c;
            f = ppm_lds<QW, ORD>(col, sCY[e]);
        }
        sFy[e] = f;
    }
#pragma unroll
    for (int m = 0; m < (XH * XW + FNT - 1) / FNT; m++) {
        const int e = tid + m * FNT;
        if (e >= XH * XW) break;
        int r = e / XW, c = e - r * XW;
        int i = i0 + c, j = j0 - 3 + r;
        T f = 0;
        if (i <= n && j <= n + 2) {
            const T *row = sQ + r * QW + c;
            f = ppm_lds<1, ORD>(row, sCX[e]);
        }
        sFx[e] = f;
    }
    {
        // faces with an edge cell upwind, on sweeps whose cross index lies
        // inside the tile (at most six per row or column): the one-sided
        // values replace the centred ones
        __syncthreads();
        for (int e = tid; e < XH * 6; e += FNT) {
            const int r = e / 6, i = edge_face_at(e - r * 6, n), c = i - i0, j = j0 - 3 + r;
            if (c < 0 || c >= XW || j < 0 || j >= n) continue;
            bool west;
            const int pe = edge_pe(i, n, west);
            const int f = r * XW + c;
            sFx[f] = ppm_edge<ORD>(sQ + r * QW + c, 1, DXA + j * P + i - 3, 1, sCX[f], pe, west);
        }
        for (int e = tid; e < YW * 6; e += FNT) {
            const int c = e / 6, j = edge_face_at(e - c * 6, n), r = j - j0, i = i0 - 3 + c;
            if (r < 0 || r >= YH || i < 0 || i >= n) continue;
            bool west;
            const int pe = edge_pe(j, n, west);
            const int f = r * YW + c;
            sFy[f] = ppm_edge<ORD>(sQy + r * QW + c, QW, DYA + (j - 3) * P + i, P, sCY[f], pe, west);
        }
    }
    __syncthreads();
    // 3. inner advective half updates
#pragma unroll
    for (int m = 0; m < (FTY * QW + FNT - 1) / FNT; m++) {
        const int e = tid + m * FNT;
        if (e >= FTY * QW) break;
        int r = e / QW, c = e - r * QW;
        int i = i0 - 3 + c, j = j0 + r;
        T v = 0;
        if (i <= n + 2 && j < n) {
            T ar = sAR[(r + 3) * QW + c];
            T y0 = sYF[r * YW + c], y1 = sYF[(r + 1) * YW + c];
            v = rdiv(sQ[(r + 3) * QW + c] * ar + y0 * sFy[r * YW + c] - y1 * sFy[(r + 1) * YW + c], ar + y0 - y1);
        }
        sQi[e] = v;
    }
#pragma unroll
    for (int m = 0; m < (QH * FTX + FNT - 1) / FNT; m++) {
        const int e = tid + m * FNT;
        if (e >= QH * FTX) break;
        int r = e / FTX, c = e - r * FTX;
        int i = i0 + c, j = j0 - 3 + r;
        T v = 0;
        if (i < n && j <= n + 2) {
            T ar = sAR[r * QW + c + 3];
            T x0 = sXF[r * XW + c], x1 = sXF[r * XW + c + 1];
            v = rdiv(sQ[r * QW + c + 3] * ar + x0 * sFx[r * XW + c] - x1 * sFx[r * XW + c + 1], ar + x0 - x1);
        }
        sQj[e] = v;
    }
    __syncthreads();
    // 4. final fluxes (in place over the outer fluxes)
    // am, ac: the old accumulator values of the face (delp epilogue)
    auto put_x = [&](int i, int c, int fi, int s, T fx, T wgt, double am, C ac) {
        const T F = (T)0.5 * (fx + sFx[s]) * wgt;
        sFx[s] = F;
        if (c < FTX || i == n) {
            if (A.FX && (!A.edges_only || i == 0 || i == n)) sto(A.FX + oc, (unsigned)fi, F);
            if (EPI == EPI_DELP) {
                sto(A.mfx + oc, (unsigned)fi, am + (double)F);
                sto(A.cxa + oc, (unsigned)fi, (C)(ac + (C)sCX[s]));
            }
        }
    };
    auto put_y = [&](int j, int r, int fi, int s, T fy, T wgt, double am, C ac) {
        const T F = (T)0.5 * (fy + sFy[s]) * wgt;
        sFy[s] = F;
        if (r < FTY || j == n) {
            if (A.FY && (!A.edges_only || j == 0 || j == n)) sto(A.FY + oc, (unsigned)fi, F);
            if (EPI == EPI_DELP) {
                sto(A.mfy + oc, (unsigned)fi, am + (double)F);
                sto(A.cya + oc, (unsigned)fi, (C)(ac + (C)sCY[s]));
            }
        }
    };
#pragma unroll
    for (int m = 0; m < N4X; m++) {
        int e = tid + m * FNT;
        if (e >= FTY * XW) break;
        int r = e / XW, c = e - r * XW;
        int i = i0 + c, j = j0 + r;
        if (i <= n && j < n && !edge_face(i, n)) {
            const int s = (r + 3) * XW + c;
            T fx = ppm_lds<1, ORD>(sQi + r * QW + c, sCX[s]);
            put_x(i, c, j * P + i, s, fx, A.mx ? (T)wx[m] : sXF[s], amx[EPI == EPI_DELP ? m : 0],
                  acx[EPI == EPI_DELP ? m : 0]);
        }
    }
    {
        // the faces with an edge cell upwind, at most six per row
        for (int e = tid; e < FTY * 6; e += FNT) {
            const int r = e / 6, i = edge_face_at(e - r * 6, n), c = i - i0, j = j0 + r;
            if (c < 0 || c >= XW || j >= n) continue;
            const int fi = j * P + i, s = (r + 3) * XW + c;
            bool west;
            const int pe = edge_pe(i, n, west);
            T fx = ppm_edge<ORD>(sQi + r * QW + c, 1, DXA + j * P + i - 3, 1, sCX[s], pe, west);
            const bool own = EPI == EPI_DELP && (c < FTX || i == n);
            put_x(i, c, fi, s, fx, MX ? (T)ldo(MX, (unsigned)fi) : sXF[s],
                  own ? ldo(A.mfx + oc, (unsigned)fi) : 0.0, own ? ldo(A.cxa + oc, (unsigned)fi) : (C)0);
        }
    }
#pragma unroll
    for (int m = 0; m < N4Y; m++) {
        int e = tid + m * FNT;
        if (e >= YH * FTX) break;
        int r = e / FTX, c = e - r * FTX;
        int i = i0 + c, j = j0 + r;
        if (i < n && j <= n && !edge_face(j, n)) {
            const int s = r * YW + c + 3;
            T fy = ppm_lds<FTX, ORD>(sQj + r * FTX + c, sCY[s]);
            put_y(j, r, j * P + i, s, fy, A.my ? (T)wy[m] : sYF[s], amy[EPI == EPI_DELP ? m : 0],
                  acy[EPI == EPI_DELP ? m : 0]);
        }
    }
    {
        // the faces with an edge cell upwind, at most six per column
        for (int e = tid; e < FTX * 6; e += FNT) {
            const int c = e / 6, j = edge_face_at(e - c * 6, n), r = j - j0, i = i0 + c;
            if (r < 0 || r >= YH || i >= n) continue;
            const int fi = j * P + i, s = r * YW + c + 3;
            bool west;
            const int pe = edge_pe(j, n, west);
            T fy = ppm_edge<ORD>(sQj + r * FTX + c, FTX, DYA + (j - 3) * P + i, P, sCY[s], pe, west);
            const bool own = EPI == EPI_DELP && (r < FTY || j == n);
            put_y(j, r, fi, s, fy, MY ? (T)ldo(MY, (unsigned)fi) : sYF[s],
                  own ? ldo(A.mfy + oc, (unsigned)fi) : 0.0, own ? ldo(A.cya + oc, (unsigned)fi) : (C)0);
        }
    }
    if constexpr (EPI == EPI_FLUX) return;
    __syncthreads();
    // 5. flux-divergence update of the cells of the tile
    const long oq = pidx(G, A.Lq, t, k);
#pragma unroll
    for (int m = 0; m < N5; m++) {
        int e = tid + m * FNT;
        if (e >= FTY * FTX) break;
        int r = e / FTX, c = e - r * FTX;
        int i = i0 + c, j = j0 + r;
        if (i >= n || j >= n) continue;
        int ci = j * P + i;
        T fw = sFx[(r + 3) * XW + c], fe = sFx[(r + 3) * XW + c + 1];
        T fs = sFy[r * YW + c + 3], fn = sFy[(r + 1) * YW + c + 3];
        T ar = sAR[(r + 3) * QW + c + 3];
        T qc = sQ[(r + 3) * QW + c + 3];
        T out;
        if constexpr (EPI == EPI_DELP) {
            out = qc + rdiv(fw - fe + fs - fn, ar);
        } else if constexpr (EPI == EPI_MASSW) {
            out = rdiv(qc * (T)pa[m] * ar + fw - fe + fs - fn, (T)pb[m] * ar);
        } else if constexpr (EPI == EPI_ADV) {
            T x0 = sXF[(r + 3) * XW + c], x1 = sXF[(r + 3) * XW + c + 1];
            T y0 = sYF[r * YW + c + 3], y1 = sYF[(r + 1) * YW + c + 3];
            out = rdiv(qc * ar + fw - fe + fs - fn, ar + x0 - x1 + y0 - y1);
        } else {
            out = (T)(((double)qc * pa[m] * (double)ar + (double)fw - (double)fe + (double)fs - (double)fn) /
                      (pb[m] * (double)ar));
        }
        sto(A.qout + oq, (unsigned)ci, out);
    }
}


template <class T, class C, class M, int EPI, int ORD>
DEVI void k_fvtp(Bk bk, Geo G, FvArgs<T, C, M> A)
{
    constexpr int FTX = FvTile<T>::X, FTY = FvTile<T>::Y;
    __shared__ FvLds<T> L;
    const int n = G.n, i0 = bk.x * FTX, j0 = bk.y * FTY;
    const bool corner = G.cube && (i0 - 3 < 0 || i0 + FTX + 2 >= n) && (j0 - 3 < 0 || j0 + FTY + 2 >= n);
    if (corner) fvtp_body<T, C, M, EPI, ORD, true>(bk, G, A, L);
    else fvtp_body<T, C, M, EPI, ORD, false>(bk, G, A, L);
}

template <class T, class C, class M, int ORD>
static void fvtp_order(const fv3_grid *g, int planes, const FvArgs<T, C, M> &a, hipStream_t st)
{
    static const char *names[] = {"k_fvtp_flux", "k_fvtp_delp", "k_fvtp_massw", "k_fvtp_adv", "k_fvtp_tracer"};
    constexpr int FTX = FvTile<T>::X, FTY = FvTile<T>::Y;
    dim3 grd((unsigned)((g->n + FTX - 1) / FTX), (unsigned)((g->n + FTY - 1) / FTY), (unsigned)planes);
    if constexpr (ORD == 7) {
        // the positive-definite order exists for the tracer transport only
        launch_fn<k_fvtp<T, C, M, EPI_TRACER, ORD>>(names[EPI_TRACER], grd, dim3(FNT), st, g->geo, a);
    } else {
        switch (a.epi) {
        case EPI_FLUX: launch_fn<k_fvtp<T, C, M, EPI_FLUX, ORD>>(names[a.epi], grd, dim3(FNT), st, g->geo, a); break;
        case EPI_DELP: launch_fn<k_fvtp<T, C, M, EPI_DELP, ORD>>(names[a.epi], grd, dim3(FNT), st, g->geo, a); break;
        case EPI_MASSW: launch_fn<k_fvtp<T, C, M, EPI_MASSW, ORD>>(names[a.epi], grd, dim3(FNT), st, g->geo, a); break;
        case EPI_ADV: launch_fn<k_fvtp<T, C, M, EPI_ADV, ORD>>(names[a.epi], grd, dim3(FNT), st, g->geo, a); break;
        default: launch_fn<k_fvtp<T, C, M, EPI_TRACER, ORD>>(names[a.epi], grd, dim3(FNT), st, g->geo, a); break;
        }
    }
}

template <class T, class C, class M>
static void fvtp_ord(const fv3_grid *g, int ord, int planes, const FvArgs<T, C, M> &a, hipStream_t st)
{
    switch (ord) {
    case 5: fvtp_order<T, C, M, 5>(g, planes, a, st); break;
    case 6: fvtp_order<T, C, M, 6>(g, planes, a, st); break;
    case 7: fvtp_order<T, C, M, 7>(g, planes, a, st); break;
    default: fvtp_order<T, C, M, 8>(g, planes, a, st); break;
    }
}

// the grid's PPM order applies to every transport of the call; the tracer
// transport takes hord_tr when that is set.  On the cube with edge_ppm the
// tile-edge instantiation runs, with the cell widths in the field's type.
template <class T, class C, class M>
static void fvtp(const fv3_grid *g, int planes, const FvArgs<T, C, M> &a, hipStream_t st)
{
    int ord = g->p.hord;
    if (a.epi == EPI_TRACER && g->p.hord_tr != 0) ord = g->p.hord_tr;
    FvArgs<T, C, M> b = a;
    if constexpr (std::is_same<T, double>::value) {
        b.dxa = g->met[M_DXA];
        b.dya = g->met[M_DYA];
    } else {
        b.dxa = g->metf[M_DXA];
        b.dya = g->metf[M_DYA];
    }
    fvtp_ord<T, C, M>(g, ord, planes, b, st);
}

// ====================================================================
// d_sw (full step bdt on one level), around the fused transport
// ====================================================================
// Courant numbers and area fluxes from the contravariant half-step C-grid
// winds (partner component: four-point mean of the other C-grid wind).  Two
// fields in, six out: bound by the stores and by latency, so a thread takes
// CRK (four, or one) consecutive layers of its point, all their loads in flight, and loads
// the metric terms once.  C192 x 79, FP32 / FP64: one layer a thread in blocks
// of 16 x 16 259 / 442 us, two 230 / 388, four 235 / 350 (32 x 8: 190 / 392,
// 64 x 4: 187 / 390), eight 243 / 330; C48 x 79 FP32: 19 us with four, 23 with
// eight (too few blocks); periodic 48 x 8 FP64, the whole call of ten
// substeps: 1117 us with one, 1147 with four.
// CORNER = false for blocks whose reads cannot reach a cube corner block
// (no view checks).
template <class B, int CRK, bool CORNER>
DEVI bool dsw_courant_body(const Geo &G, const Mets<B> &M, B bdt, const B *uc, const B *vc, int t, int k0, int i, int j,
                           B *ut, B *vt, B *crx, B *cry, B *xfx, B *yfx)
{
    const int n = G.n, k1 = min(k0 + CRK, G.nz);
    const bool fx = i >= 0 && i <= n && j >= -3 && j <= n + 2, fy = i >= -3 && i <= n + 2 && j >= 0 && j <= n;
    const B *dxa = MP(M, M_DXA), *dya = MP(M, M_DYA);
    bool bad = false;
    if (fx) {
        const B su = AT(MP(M, M_SIN_U), i, j), cu = AT(MP(M, M_COS_U), i, j), dy = AT(MP(M, M_DY), i, j);
        const B dw = CORNER ? pvx(G, dxa, dya, SC, i - 1, j, 0, false) : AT(dxa, i - 1, j);
        const B de = CORNER ? pvx(G, dxa, dya, SC, i, j, 0, false) : AT(dxa, i, j);
#pragma unroll
        for (int q = 0; q < CRK; q++) {
            const long o = pidx(G, G.nz, t, min(k0 + q, k1 - 1));
            const B *UC = uc + o, *VC = vc + o;
            B vb;
            if constexpr (CORNER)
                vb = (B)0.25 * (pvy(G, UC, VC, SY, i - 1, j, 0, true) + pvy(G, UC, VC, SY, i, j, 0, true) +
                                pvy(G, UC, VC, SY, i - 1, j + 1, 0, true) + pvy(G, UC, VC, SY, i, j + 1, 0, true));
            else
                vb = (B)0.25 * (AT(VC, i - 1, j) + AT(VC, i, j) + AT(VC, i - 1, j + 1) + AT(VC, i, j + 1));
            B uu = rdiv(AT(UC, i, j) - vb * cu, su * su);
            B da = uu > 0 ? dw : de;
            B cr = rdiv(bdt * uu, da);
            if (k0 + q < k1) {
                AT(ut + o, i, j) = uu;
                AT(crx + o, i, j) = cr;
                AT(xfx + o, i, j) = bdt * uu * su * dy;
                bad |= fabs((double)cr) > 1.0;
            }
        }
    }
    if (fy) {
        const B sv_ = AT(MP(M, M_SIN_V), i, j), cv = AT(MP(M, M_COS_V), i, j), dx = AT(MP(M, M_DX), i, j);
        const B ds = CORNER ? pvy(G, dxa, dya, SC, i, j - 1, 1, false) : AT(dya, i, j - 1);
        const B dn = CORNER ? pvy(G, dxa, dya, SC, i, j, 1, false) : AT(dya, i, j);
#pragma unroll
        for (int q = 0; q < CRK; q++) {
            const long o = pidx(G, G.nz, t, min(k0 + q, k1 - 1));
            const B *UC = uc + o, *VC = vc + o;
            B ub;
            if constexpr (CORNER)
                ub = (B)0.25 * (pvx(G, UC, VC, SX, i, j - 1, 1, true) + pvx(G, UC, VC, SX, i + 1, j - 1, 1, true) +
                                pvx(G, UC, VC, SX, i, j, 1, true) + pvx(G, UC, VC, SX, i + 1, j, 1, true));
            else
                ub = (B)0.25 * (AT(UC, i, j - 1) + AT(UC, i + 1, j - 1) + AT(UC, i, j) + AT(UC, i + 1, j));
            B vv = rdiv(AT(VC, i, j) - ub * cv, sv_ * sv_);
            B da = vv > 0 ? ds : dn;
            B cr = rdiv(bdt * vv, da);
            if (k0 + q < k1) {
                AT(vt + o, i, j) = vv;
                AT(cry + o, i, j) = cr;
                AT(yfx + o, i, j) = bdt * vv * sv_ * dx;
                bad |= fabs((double)cr) > 1.0;
            }
        }
    }
    return bad;
}
template <class B>
DEVI void k_dsw_courant(KARGS, Geo G, Mets<B> M, int layers, B bdt, const B *uc, const B *vc, B *ut, B *vt,
                              B *crx, B *cry, B *xfx, B *yfx, int *flags)
{
    KBEGIN((G.nz + layers - 1) / layers);
    // the block's reads span its points +-1 in both directions; corner views
    // exist only outside [0, n - 1] in both
    const int i0 = ib + (int)(bk.x * blockDim.x) - 1, i1 = i0 + (int)blockDim.x + 1;
    const int j0 = jlo + (int)(bk.y * blockDim.y) - 1, j1 = j0 + (int)blockDim.y + 1;
    const bool corner = G.cube && (i0 < 0 || i1 >= G.n) && (j0 < 0 || j1 >= G.n);
    bool bad;
    if (layers == 1) {
        if (corner) bad = dsw_courant_body<B, 1, true>(G, M, bdt, uc, vc, t, k, i, j, ut, vt, crx, cry, xfx, yfx);
        else bad = dsw_courant_body<B, 1, false>(G, M, bdt, uc, vc, t, k, i, j, ut, vt, crx, cry, xfx, yfx);
    } else {
        if (corner) bad = dsw_courant_body<B, 4, true>(G, M, bdt, uc, vc, t, k * 4, i, j, ut, vt, crx, cry, xfx, yfx);
        else bad = dsw_courant_body<B, 4, false>(G, M, bdt, uc, vc, t, k * 4, i, j, ut, vt, crx, cry, xfx, yfx);
    }
    if (bad) atomicOr(flags, 1);
}

// absolute vorticity at cells from the D-grid circulation, and the kinetic
// energy at corners (D-grid u upwinded along x and v along y by PPM with the
// corner displacements of the contravariant C-grid winds)
template <class B, int ORD>
DEVI void k_dsw_omke(KARGS, Geo G, Mets<B> M, B bdt, B d2, B dd, B damin, const B *u, const B *v,
                           const B *ut, const B *vt, const B *hd, B hc, B *om, B *ke)
{
    int i, j;
    if constexpr (sizeof(B) == 4) {
        // FP32 (bound by its arithmetic): launched over the range flattened
        // by rows, so that no wavefront is mostly idle at the range's ends
        const int w = ihi - ilo + 1, p = (int)(bk.x * blockDim.x + threadIdx.x);
        if (p >= w * (jhi - jlo + 1)) return;
        j = jlo + p / w;
        i = ilo + p % w;
    } else {
        i = ib + (int)(bk.x * blockDim.x + threadIdx.x);
        j = jlo + (int)(bk.y * blockDim.y + threadIdx.y);
        if (i < ilo || i > ihi || j > jhi) return;
    }
    const int t = (int)bk.z / G.nz, k = (int)bk.z % G.nz;
    int n = G.n;
    long o = pidx(G, G.nz, t, k);
    const B *U = u + o, *V = v + o;
    const B *dx = MP(M, M_DX), *dy = MP(M, M_DY);
    if (!in_corner(G, SC, i, j) && i <= n + 2 && j <= n + 2)
        AT(om + o, i, j) = AT(MP(M, M_FC), i, j) + rdiv(AT(U, i, j) * AT(dx, i, j) - AT(U, i, j + 1) * AT(dx, i, j + 1) -
                                                         AT(V, i, j) * AT(dy, i, j) + AT(V, i + 1, j) * AT(dy, i + 1, j),
                                                     AT(MP(M, M_AREA), i, j));
    if (i >= 0 && i <= n && j >= 0 && j <= n) {
        B ub = (B)0.5 * bdt * (AT(ut + o, i, j - 1) + AT(ut + o, i, j));
        B vb = (B)0.5 * bdt * (AT(vt + o, i - 1, j) + AT(vt + o, i, j));
        B cu = rdiv(ub, AT(dx, ub > 0 ? i - 1 : i, j));
        B cv = rdiv(vb, AT(dy, i, vb > 0 ? j - 1 : j));
        B uu = ppm6<ORD>(AT(U, i - 3, j), AT(U, i - 2, j), AT(U, i - 1, j), AT(U, i, j), AT(U, i + 1, j), AT(U, i + 2, j), cu);
        B vv = ppm6<ORD>(AT(V, i, j - 3), AT(V, i, j - 2), AT(V, i, j - 1), AT(V, i, j), AT(V, i, j + 1), AT(V, i, j + 2), cv);
        B kev = (B)0.5 * (ub * uu + vb * vv);
        if (d2 > (B)0 || dd > (B)0) {
            // del-2 divergence damping: minus nu times the divergence of the
            // D-grid winds over the corner's dual cell (half weights next to
            // the missing cell at a cube vertex), nu = damin times d2, raised
            // by the Smagorinsky magnitude dd sqrt(DT^2 + DS^2) up to 0.2
            B ws = 1, wn = 1, ww = 1, we = 1;
            if (is_vertex(G, i, j)) {
                if (j == 0) ws = 0.5; else wn = 0.5;
                if (i == 0) ww = 0.5; else we = 0.5;
            }
            const B *dxc = MP(M, M_DXC), *dyc = MP(M, M_DYC);
            B rac = AT(MP(M, M_RAREA_C), i, j);
            B fe = we * AT(U, i, j) * AT(dyc, i, j), fw = ww * AT(U, i - 1, j) * AT(dyc, i - 1, j);
            B fn = wn * AT(V, i, j) * AT(dxc, i, j), fs = ws * AT(V, i, j - 1) * AT(dxc, i, j - 1);
            B c2 = d2;
            if (dd > (B)0) {
                // tension at the corner; shear of the stored cells around it
                B ten = (fe - fw - fn + fs) * rac, sh = 0;
                int cnt = 0;
                const B *ra = MP(M, M_RAREA);
                for (int cj = j - 1; cj <= j; cj++)
                    for (int ci = i - 1; ci <= i; ci++) {
                        if (in_corner(G, SC, ci, cj)) continue;
                        sh += (AT(V, ci + 1, cj) * AT(dy, ci + 1, cj) - AT(V, ci, cj) * AT(dy, ci, cj) +
                               AT(U, ci, cj + 1) * AT(dx, ci, cj + 1) - AT(U, ci, cj) * AT(dx, ci, cj)) *
                              AT(ra, ci, cj);
                        cnt++;
                    }
                sh /= (B)cnt;
                B cs = dd * sqrt(ten * ten + sh * sh);
                cs = cs < (B)0.2 ? cs : (B)0.2;
                c2 = cs > c2 ? cs : c2;
            }
            kev -= c2 * damin * (fe - fw + fn - fs) * rac;
        }
        // higher-order damping: hc = (-1)^(nord+1) nu_n times the divergence
        // after nord corner Laplacians
        if (hd) kev += hc * AT(hd + o, i, j);
        AT(ke + o, i, j) = kev;
    }
}

// Edge-flux fix-up on the cube, one thread per (cell next to a tile edge,
// level): each of the cell's faces on the edge takes the mean of our flux and
// the neighbour tile's copy (mapped onto our direction); the cell takes the
// difference.  After d_sw: mass fluxes FXm/FYm (delp), content fluxes of pt
// and w, the committed delp, pt, w and the mass-flux accumulators.
template <class B>
DEVI B edge_mean_delta(const Geo &G, const EdgeCell &c, int q, int k, const B *FX, const B *FY)
{
    const B *own = c.arr[q] == 0 ? FX : FY, *par = c.parr[q] == 0 ? FX : FY;
    const B fo = own[pidx(G, G.nz, c.t, k) + c.off[q]];
    const B fp = (B)c.spar[q] * par[pidx(G, G.nz, c.pt[q], k) + c.poff[q]];
    return (B)0.5 * (fo + fp) - fo;
}

// Tile-edge kinetic energy (edge_ppm): at the corners whose wind sweeps have
// an edge cell upwind (i or j in 0, 1, 2, n-2, n-1, n) the upwinded winds take
// the one-sided face values, the widths being the face lengths dx (dy); the
// difference from the centred values k_dsw_omke used is added to ke.  One
// thread per corner of the six lines of each direction (corners on both a
// column and a row line counted once), levels in y, tiles in z.
template <class B, int ORD>
DEVI void k_ke_edge(Bk bk, Geo G, Mets<B> M, B bdt, const B *u, const B *v, const B *ut, const B *vt, B *ke)
{
    const int n = G.n, e = (int)(bk.x * blockDim.x + threadIdx.x), k = (int)bk.y, t = (int)bk.z;
    int i, j;
    if (e < 6 * (n + 1)) {
        // the six edge columns of one row are neighbouring threads
        j = e / 6;
        i = edge_face_at(e - 6 * j, n);
    } else {
        const int e2 = e - 6 * (n + 1);
        if (e2 >= 6 * (n - 5)) return;
        const int q = e2 / (n - 5);
        i = 3 + e2 - q * (n - 5);
        j = edge_face_at(q, n);
    }
    const long o = pidx(G, G.nz, t, k);
    const B *U = u + o, *V = v + o;
    const B *dx = MP(M, M_DX), *dy = MP(M, M_DY);
    B d = 0;
    bool west;
    if (edge_face(i, n)) {
        const B ub = (B)0.5 * bdt * (AT(ut + o, i, j - 1) + AT(ut + o, i, j));
        const B cu = rdiv(ub, AT(dx, ub > 0 ? i - 1 : i, j));
        const int pe = edge_pe(i, n, west);
        const B ue = ppm_edge<ORD>(&AT(U, i - 3, j), 1, &AT(dx, i - 3, j), 1, cu, pe, west);
        const B uc = ppm6<ORD>(AT(U, i - 3, j), AT(U, i - 2, j), AT(U, i - 1, j), AT(U, i, j), AT(U, i + 1, j),
                               AT(U, i + 2, j), cu);
        d += ub * (ue - uc);
    }
    if (edge_face(j, n)) {
        const B vb = (B)0.5 * bdt * (AT(vt + o, i - 1, j) + AT(vt + o, i, j));
        const B cv = rdiv(vb, AT(dy, i, vb > 0 ? j - 1 : j));
        const int pe = edge_pe(j, n, west);
        const B ve = ppm_edge<ORD>(&AT(V, i, j - 3), (int)G.pitch, &AT(dy, i, j - 3), (int)G.pitch, cv, pe, west);
        const B vc = ppm6<ORD>(AT(V, i, j - 3), AT(V, i, j - 2), AT(V, i, j - 1), AT(V, i, j), AT(V, i, j + 1),
                               AT(V, i, j + 2), cv);
        d += vb * (ve - vc);
    }
    AT(ke + o, i, j) += (B)0.5 * d;
}

template <class B>
DEVI void k_edgefix_dsw(Bk bk, Geo G, const EdgeCell *__restrict__ cells, int count, const B *area,
                        const B *FXm, const B *FYm, const B *FXp, const B *FYp, const B *FXw, const B *FYw,
                        B *delp, B *pt, B *w, double *mfx, double *mfy)
{
    const int e = (int)(bk.x * blockDim.x + threadIdx.x);
    if (e >= count) return;
    const int k = (int)bk.y;
    const EdgeCell c = cells[e];
    B dM = 0, dP = 0, dW = 0;
    for (int q = 0; q < c.nf; q++) {
        const B em = edge_mean_delta(G, c, q, k, FXm, FYm);
        dM += (B)c.sin[q] * em;
        dP += (B)c.sin[q] * edge_mean_delta(G, c, q, k, FXp, FYp);
        dW += (B)c.sin[q] * edge_mean_delta(G, c, q, k, FXw, FYw);
        double *acc = c.arr[q] == 0 ? mfx : mfy;
        acc[pidx(G, G.nz, c.t, k) + c.off[q]] += (double)em;
    }
    const long o = pidx(G, G.nz, c.t, k) + c.cell;
    const B a = area[pidx(G, 1, c.t, 0) + c.cell];
    const B d0 = delp[o], d1 = d0 + dM / a;
    pt[o] = (pt[o] * d0 * a + dP) / (d1 * a);
    w[o] = (w[o] * d0 * a + dW) / (d1 * a);
    delp[o] = d1;
}

// ... and after a tracer sub-cycle: tracer fluxes, the sub-cycle's new mass dp2.
template <class B>
DEVI void k_edgefix_q(Bk bk, Geo G, const EdgeCell *__restrict__ cells, int count, const B *area, const B *FX,
                      const B *FY, const double *dp2, B *qf)
{
    const int e = (int)(bk.x * blockDim.x + threadIdx.x);
    if (e >= count) return;
    const int k = (int)bk.y;
    const EdgeCell c = cells[e];
    B dQ = 0;
    for (int q = 0; q < c.nf; q++) dQ += (B)c.sin[q] * edge_mean_delta(G, c, q, k, FX, FY);
    const long o = pidx(G, G.nz, c.t, k) + c.cell;
    qf[o] = qf[o] + (B)((double)dQ / (dp2[o] * (double)area[pidx(G, 1, c.t, 0) + c.cell]));
}

// Divergence at corner (i, j) of a D-grid pair (U on y-faces, V on x-faces)
// over the corner's dual cell: normal components through its four edges
// times their lengths over the dual area, half weights for the two edges
// next to the missing cell at a cube vertex.
template <class B>
DEVI B corner_div_at(const Geo &G, const Mets<B> &M, const B *U, const B *V, int t, int i, int j)
{
    B ws = 1, wn = 1, ww = 1, we = 1;
    if (is_vertex(G, i, j)) {
        if (j == 0) ws = 0.5; else wn = 0.5;
        if (i == 0) ww = 0.5; else we = 0.5;
    }
    const B *dxc = MP(M, M_DXC), *dyc = MP(M, M_DYC);
    return (we * AT(U, i, j) * AT(dyc, i, j) - ww * AT(U, i - 1, j) * AT(dyc, i - 1, j) +
            wn * AT(V, i, j) * AT(dxc, i, j) - ws * AT(V, i, j - 1) * AT(dxc, i, j - 1)) *
           AT(MP(M, M_RAREA_C), i, j);
}

// Higher-order divergence damping: the corner divergence of the D-grid
// winds (corners 0..n of every level) ...
template <class B>
DEVI void k_cdiv(KARGS, Geo G, Mets<B> M, const B *u, const B *v, B *dg)
{
    KBEGIN(G.nz);
    long o = pidx(G, G.nz, t, k);
    AT(dg + o, i, j) = corner_div_at(G, M, u + o, v + o, t, i, j);
}

// ... and the corner Laplacian of a corner field whose halo is filled: the
// corner divergence of its gradient along the cell edges, (D(i+1,j) -
// D(i,j)) / dx on y-faces and (D(i,j+1) - D(i,j)) / dy on x-faces.
template <class B>
DEVI void k_clap(KARGS, Geo G, Mets<B> M, const B *d, B *out)
{
    KBEGIN(G.nz);
    long o = pidx(G, G.nz, t, k);
    const B *D = d + o, *rdx = MP(M, M_RDX), *rdy = MP(M, M_RDY);
    const B c = AT(D, i, j);
    const B ge = (AT(D, i + 1, j) - c) * AT(rdx, i, j), gw = (c - AT(D, i - 1, j)) * AT(rdx, i - 1, j);
    const B gn = (AT(D, i, j + 1) - c) * AT(rdy, i, j), gs = (c - AT(D, i, j - 1)) * AT(rdy, i, j - 1);
    B ws = 1, wn = 1, ww = 1, we = 1;
    if (is_vertex(G, i, j)) {
        if (j == 0) ws = 0.5; else wn = 0.5;
        if (i == 0) ww = 0.5; else we = 0.5;
    }
    const B *dxc = MP(M, M_DXC), *dyc = MP(M, M_DYC);
    AT(out + o, i, j) = (we * ge * AT(dyc, i, j) - ww * gw * AT(dyc, i - 1, j) + wn * gn * AT(dxc, i, j) -
                         ws * gs * AT(dxc, i, j - 1)) *
                        AT(MP(M, M_RAREA_C), i, j);
}

// D-grid wind update from kinetic-energy differences and vorticity fluxes.
// Optional del-2 vorticity damping (nuv > 0): the diffusive flux of the
// relative vorticity (om - f) across each face joins the vorticity flux, so
// u gains nuv (w(i, j-1) - w(i, j)) / dyc and v loses nuv (w(i-1, j) - w(i, j)) / dxc.
template <class B>
DEVI void k_dsw_update(KARGS, Geo G, Mets<B> M, const B *ke, const B *VX, const B *VY,
                             const B *om, B nuv, B *u, B *v)
{
    KBEGIN(G.nz);
    int n = G.n;
    long o = pidx(G, G.nz, t, k);
    const B *KE = ke + o;
    B du = 0, dv = 0;
    if (nuv > (B)0) {
        const B *OM = om + o, *fc = MP(M, M_FC);
        const B wc = AT(OM, i, j) - AT(fc, i, j);
        if (i < n) du = nuv * ((AT(OM, i, j - 1) - AT(fc, i, j - 1)) - wc) * AT(MP(M, M_RDYC), i, j);
        if (j < n) dv = -nuv * ((AT(OM, i - 1, j) - AT(fc, i - 1, j)) - wc) * AT(MP(M, M_RDXC), i, j);
    }
    if (i < n) AT(u + o, i, j) = AT(u + o, i, j) + (AT(KE, i, j) - AT(KE, i + 1, j) + AT(VY + o, i, j)) * AT(MP(M, M_RDX), i, j) + du;
    if (j < n) AT(v + o, i, j) = AT(v + o, i, j) + (AT(KE, i, j) - AT(KE, i, j + 1) - AT(VX + o, i, j)) * AT(MP(M, M_RDY), i, j) + dv;
}

// ====================================================================
// dz_d: the interface heights (kept from substep to substep, column.hip) are
// transported by fv_tp_2d (EPI_ADV, interface averaged Courant numbers),
// surface fixed.
// ====================================================================
// Halo of the interface heights.  A halo column stands on the surface height
// the caller's phis holds at that halo point, which is the neighbour cell's
// where phis is consistent.  delz, where given, is exchanged with them: nothing
// here reads its halo, the caller may.
DEVI void k_halo_z(Bk bk, Geo G, const HaloEnt *__restrict__ plan, int count, const double *phis, double *z, int L,
                   double *delz)
{
    const int e = (int)(bk.x * blockDim.x + threadIdx.x);
    if (e >= count) return;
    const int k = (int)bk.y;
    const HaloEnt h = plan[e];
    double v = z[pidx(G, L, h.st, k) + h.si];
    if (phis) {
        const double zs = phis[pidx(G, 1, h.st, 0) + h.si] / GRAV, zd = phis[pidx(G, 1, h.dt, 0) + h.di] / GRAV;
        if (zs != zd) v = (v - zs) + zd;
    }
    z[pidx(G, L, h.dt, k) + h.di] = v;
    if (delz && k < L - 1) delz[pidx(G, L - 1, h.dt, k) + h.di] = delz[pidx(G, L - 1, h.st, k) + h.si];
}

// Mixed precision: the heights travel as FP32 deviations from a reference
// per (tile, interface), the height at cell (0, 0).  The transport is exactly
// translation-equivariant (PPM faces, advective inner and outer updates), so
// only the deviations' rounding enters, not that of the full height.  The
// thread of cell (0, 0) stores the reference.
DEVI void k_zdev(KARGS, Geo G, const double *z, double *zref, float *zd)
{
    KBEGIN(G.nz + 1);
    if (in_corner(G, SC, i, j)) return;
    const long o = pidx(G, G.nz + 1, t, k);
    const double zr = AT(z + o, 0, 0);
    AT(zd + o, i, j) = (float)(AT(z + o, i, j) - zr);
    if (i == 0 && j == 0) zref[t * (G.nz + 1) + k] = zr;
}

// The substep commits the transported fields in the second column solve;
// these two do it where a debug call stops before it.
template <class B>
DEVI void k_commit(KARGS, Geo G, const B *dn, const B *pn, const B *wn, B *delp, B *pt, B *w)
{
    KBEGIN(G.nz);
    const long o = pidx(G, G.nz, t, k);
    AT(delp + o, i, j) = AT(dn + o, i, j);
    AT(pt + o, i, j) = AT(pn + o, i, j);
    AT(w + o, i, j) = AT(wn + o, i, j);
}
DEVI void k_delz_from_zdev(KARGS, Geo G, const float *zn, const double *zref, const double *phis, double *delz)
{
    KBEGIN(G.nz);
    int nz = G.nz;
    const double *zr = zref + t * (nz + 1);
    double top = zr[k] + (double)AT(zn + pidx(G, nz + 1, t, k), i, j);
    double below = k == nz - 1 ? (phis ? AT(phis + pidx(G, 1, t, 0), i, j) / GRAV : 0.0)
                               : zr[k + 1] + (double)AT(zn + pidx(G, nz + 1, t, k + 1), i, j);
    AT(delz + pidx(G, nz, t, k), i, j) = below - top;
}

DEVI void k_delz_from_zh(KARGS, Geo G, const double *zn, const double *phis, double *delz)
{
    KBEGIN(G.nz);
    int nz = G.nz;
    double below = k == nz - 1 ? (phis ? AT(phis + pidx(G, 1, t, 0), i, j) / GRAV : 0.0)
                               : AT(zn + pidx(G, nz + 1, t, k + 1), i, j);
    AT(delz + pidx(G, nz, t, k), i, j) = below - AT(zn + pidx(G, nz + 1, t, k), i, j);
}

// ====================================================================
// utilities: fills, copies, finiteness check, tracer helpers, reductions
// ====================================================================
template <class T>
DEVI void k_fill(Bk bk, T *p, long count, T val)
{
    long e = (long)bk.x * blockDim.x + threadIdx.x;
    if (e < count) p[e] = val;
}
template <class TS, class TD>
DEVI void k_copy(Bk bk, const TS *s, TD *d, long count)
{
    long e = (long)bk.x * blockDim.x + threadIdx.x;
    if (e < count) d[e] = (TD)s[e];
}
template <class T>
static void fill(T *p, long count, T val, hipStream_t st)
{
    launch_fn<k_fill<T>>("k_fill", dim3((unsigned)((count + 255) / 256)), dim3(256), st, p, count, val);
}
template <class TS, class TD>
static void copy(const TS *s, TD *d, long count, hipStream_t st)
{
    launch_fn<k_copy<TS, TD>>("k_copy", dim3((unsigned)((count + 255) / 256)), dim3(256), st, s, d, count);
}

template <class T>
DEVI void k_check_finite(KARGS, Geo G, int L, const T *f, int *flags)
{
    KBEGIN(L);
    if (!isfinite((double)AT(f + pidx(G, L, t, k), i, j))) atomicOr(flags + 1, 1);
}

// tracer: area fluxes from the accumulated Courant numbers, scaled by 1/nsplt
// (and the mass fluxes where mxs, mys are given)
template <class B>
DEVI void k_tracer_flux(KARGS, Geo G, MetD M, double rs, const B *cx, const B *cy,
                              const double *mfx, const double *mfy, B *crs, B *crys, B *xfx,
                              B *yfx, double *mxs, double *mys)
{
    KBEGIN(G.nz);
    int n = G.n;
    long o = pidx(G, G.nz, t, k);
    const double *dxa = MP(M, M_DXA), *dya = MP(M, M_DYA);
    if (i >= 0 && i <= n && j >= -3 && j <= n + 2) {
        double c = (double)AT(cx + o, i, j);
        int up = c > 0 ? i - 1 : i;
        AT(xfx + o, i, j) = (B)(c * pvx(G, dxa, dya, SC, up, j, 0, false) * AT(MP(M, M_DY), i, j) *
                                AT(MP(M, M_SIN_U), i, j) / rs);
        AT(crs + o, i, j) = (B)(c / rs);
        if (mxs) AT(mxs + o, i, j) = AT(mfx + o, i, j) / rs;
    }
    if (i >= -3 && i <= n + 2 && j >= 0 && j <= n) {
        double c = (double)AT(cy + o, i, j);
        int up = c > 0 ? j - 1 : j;
        AT(yfx + o, i, j) = (B)(c * pvy(G, dxa, dya, SC, i, up, 1, false) * AT(MP(M, M_DX), i, j) *
                                AT(MP(M, M_SIN_V), i, j) / rs);
        AT(crys + o, i, j) = (B)(c / rs);
        if (mys) AT(mys + o, i, j) = AT(mfy + o, i, j) / rs;
    }
}

// interior of up to four fields, plane z of field z / planes
template <class B>
DEVI void k_copy_back(KARGS, Geo G, int planes, FieldSet<B> src, FieldSet<B> dst)
{
    KBEGIN(planes);   // t: field, k: plane
    const B *a = t == 0 ? src.p[0] : t == 1 ? src.p[1] : t == 2 ? src.p[2] : src.p[3];
    B *b = t == 0 ? dst.p[0] : t == 1 ? dst.p[1] : t == 2 ? dst.p[2] : dst.p[3];
    const long o = G.off0 + (long)k * G.lev;
    AT(b + o, i, j) = AT(a + o, i, j);
}

DEVI void k_tracer_dp(KARGS, Geo G, MetD M, const double *dp1, const double *mxs,
                            const double *mys, double *dp2)
{
    KBEGIN(G.nz);
    long o = pidx(G, G.nz, t, k);
    AT(dp2 + o, i, j) = AT(dp1 + o, i, j) + (AT(mxs + o, i, j) - AT(mxs + o, i + 1, j) + AT(mys + o, i, j) -
                                             AT(mys + o, i, j + 1)) /
                                                AT(MP(M, M_AREA), i, j);
}

// maximum that keeps a NaN (fmax drops it), so a non-finite Courant number
// reaches the host's sub-cycle count
DEVI double nanmax(double a, double b) { return (a != a || a > b) ? a : b; }

// max |cx|, |cy| over the interior faces: block maximum, one atomic per block
template <class B>
__global__ void k_absmax(int ilo, int ihi, int jlo, int jhi, Geo G, const B *cx, const B *cy, unsigned long long *out)
{
    // each block covers its (i, j) patch on every gridDim.z-th plane, so that
    // only a few thousand blocks meet at the one atomic
    __shared__ double sm[256];
    int tid = threadIdx.y * blockDim.x + threadIdx.x;
    int i = ilo + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    int j = jlo + (int)(blockIdx.y * blockDim.y + threadIdx.y);
    double m = 0.0;
    if (i <= ihi && j <= jhi) {
        int n = G.n, planes = G.T * G.nz;
        for (int z = (int)blockIdx.z; z < planes; z += (int)gridDim.z) {
            int t = z / G.nz, k = z % G.nz;
            long o = pidx(G, G.nz, t, k);
            if (j < n) m = nanmax(m, fabs((double)AT(cx + o, i, j)));
            if (i < n) m = nanmax(m, fabs((double)AT(cy + o, i, j)));
        }
    }
    sm[tid] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) sm[tid] = nanmax(sm[tid], sm[tid + w]);
        __syncthreads();
    }
    // non-negative doubles order like their bit patterns, and a NaN's bits
    // lie above those of +inf, so a NaN survives the atomic too
    if (tid == 0) atomicMax(out, (unsigned long long)__double_as_longlong(sm[0]));
}

// Neumaier-compensated sums: each thread sums its column over levels in a
// fixed order, then the block combines pairs (s, c) with Neumaier additions,
// one partial per block and field; one thread per field adds the partials in
// block order.
DEVI void neu_add(double &s, double &c, double x)
{
    const double t = s + x;
    const bool big = fabs(s) >= fabs(x);
    c += ((big ? s : x) - t) + (big ? x : s);
    s = t;
}

// Up to MNF sums share one pass (delp and the cell mass are read and formed
// once for all): field f is delp alone (null pointer) or p[f] times it.  The
// values of four levels are loaded ahead of their additions.  Bound by the
// reads: C192 x 79 mixed, six sums: six passes of 75 us -> one of 103.
constexpr int MNF = 6;
template <class B>
struct MassFields {
    const B *p[MNF];
    int nf;
};
template <class B>
__global__ void __launch_bounds__(256) k_mass_partial(int ilo, int ihi, int jlo, int jhi, Geo G, MetD M,
                                                      const B *delp, MassFields<B> F, double *part)
{
    // a product fused into a compensated addition would leave its error term wrong
#pragma clang fp contract(off)
    __shared__ double ss[MNF][256], sc[MNF][256];
    int tid = threadIdx.y * blockDim.x + threadIdx.x;
    int i = ilo + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    int j = jlo + (int)(blockIdx.y * blockDim.y + threadIdx.y);
    int t = blockIdx.z;
    double s[MNF], c[MNF];
#pragma unroll
    for (int f = 0; f < MNF; f++) s[f] = c[f] = 0.0;
    if (i <= ihi && j <= jhi) {
        const double ar = AT(MP(M, M_AREA), i, j);
        constexpr int U = 4;
        for (int k0 = 0; k0 < G.nz; k0 += U) {
            B d[U], v[MNF][U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const long o = pidx(G, G.nz, t, min(k0 + u, G.nz - 1));
                d[u] = AT(delp + o, i, j);
#pragma unroll
                for (int f = 0; f < MNF; f++)
                    if (f < F.nf && F.p[f]) v[f][u] = AT(F.p[f] + o, i, j);
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (k0 + u >= G.nz) break;
                const double m = (double)d[u] * ar;
#pragma unroll
                for (int f = 0; f < MNF; f++)
                    if (f < F.nf) neu_add(s[f], c[f], F.p[f] ? (double)v[f][u] * m : m);
            }
        }
    }
#pragma unroll
    for (int f = 0; f < MNF; f++) {
        ss[f][tid] = s[f];
        sc[f][tid] = c[f];
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) {
            for (int f = 0; f < F.nf; f++) {
                double a = ss[f][tid], ac = sc[f][tid] + sc[f][tid + w];
                neu_add(a, ac, ss[f][tid + w]);
                ss[f][tid] = a;
                sc[f][tid] = ac;
            }
        }
        __syncthreads();
    }
    if (tid < F.nf) {
        const long nb = (long)gridDim.x * gridDim.y * gridDim.z;
        const long b = ((long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        part[2 * (nb * tid + b)] = ss[tid][0];
        part[2 * (nb * tid + b) + 1] = sc[tid][0];
    }
}

// The block partials of one field per block, combined in block order: the sums
// s_i, one addition each after the other, the errors e_i of these additions,
// independent of each other once the sums are known, and the compensation c,
// two additions each.  One thread does the sums of a batch of partials, another
// the compensation of the batch two before, two wavefronts the errors of the one
// between.  Every value is that of the plain loop.  Bound by the latency of the
// additions.  One thread doing all of it / this, the whole call: two sums of C768
// x 3 (13824 partials) 423 / 223 us, of 1024 x 1024 x 2 136 / 86; six of C192 x 79
// 121 / 113.
constexpr int MFB = 256;   // partials per batch
__global__ void __launch_bounds__(256) k_mass_final(const double *part, long np, double *out)
{
#pragma clang fp contract(off)
    __shared__ double px[4][MFB], pc[4][MFB], ps[2][MFB + 1], pe[2][MFB];
    const double *p = part + 2 * np * blockIdx.x;
    const int tid = (int)threadIdx.x, nb = (int)((np + MFB - 1) / MFB);
    double s = 0.0, c = 0.0;   // thread 0: s; thread 64: c
    // partials past the last one are zeros, which change neither sum nor compensation
    auto load = [&](int b, int i) {
        const long e = (long)b * MFB + i;
        px[b & 3][i] = e < np ? p[2 * e] : 0.0;
        pc[b & 3][i] = e < np ? p[2 * e + 1] : 0.0;
    };
    load(0, tid);
    __syncthreads();
    // partials of a batch, up to the next multiple of 16
    auto count = [&](int b) { return (int)(np - (long)b * MFB < MFB ? (np - (long)b * MFB + 15) / 16 * 16 : MFB); };
    for (int b = 0; b < nb + 2; b++) {
        if (tid == 0 && b < nb) {
            const double *x = px[b & 3];
            double *o = ps[b & 1];
            const int m = count(b);
            for (int i = 0; i < m; i += 16) {
                double v[16];
#pragma unroll
                for (int q = 0; q < 16; q++) v[q] = x[i + q];
#pragma unroll
                for (int q = 0; q < 16; q++) {
                    o[i + q] = s;
                    s = s + v[q];
                }
            }
            o[m] = s;
        }
        if (tid == 64 && b >= 2) {
            const double *k = pc[(b - 2) & 3], *e = pe[b & 1];
            const int m = count(b - 2);
            for (int i = 0; i < m; i += 8) {
                double v[8], w[8];
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    v[q] = k[i + q];
                    w[q] = e[i + q];
                }
#pragma unroll
                for (int q = 0; q < 8; q++) c = (c + v[q]) + w[q];
            }
        }
        if (tid >= 128) {
            for (int i = tid - 128; i < MFB; i += 128) {
                if (b + 1 < nb) load(b + 1, i);
                if (b >= 1 && b <= nb && i < count(b - 1)) {
                    const double x = px[(b - 1) & 3][i], s0 = ps[(b - 1) & 1][i], t = ps[(b - 1) & 1][i + 1];
                    const bool big = fabs(s0) >= fabs(x);
                    pe[(b - 1) & 1][i] = ((big ? s0 : x) - t) + (big ? x : s0);
                }
            }
        }
        __syncthreads();
    }
    if (tid == 64) px[0][0] = c;
    __syncthreads();
    if (tid == 0) out[blockIdx.x] = s + px[0][0];
}

// ====================================================================
// Workspace carve-up
// ====================================================================
template <class B>
struct Work {
    // bulk layer fields
    B *ax, *ay, *delpc, *ptc, *wc, *ke;
    B *ut, *vt, *crx, *cry, *xfx, *yfx, *FX, *FY, *VX, *VY, *dn, *pn, *wn, *om, *qo;
    // FP64 fields
    double *s1, *s2, *dp1, *dp2, *mxs, *mys;
    double *pkc, *gz, *zh, *zn;   // interfaces
    unsigned long long *umax;
    double *part;
};

static long part_count(const fv3_grid *g)
{
    long bx = (g->n + 63) / 64, by = (g->n + 3) / 4;
    return bx * by * g->T;
}

template <class B>
static size_t carve(const fv3_grid *g, char *base, Work<B> *w)
{
    long el = alloc_elems(g, g->nz), ei = alloc_elems(g, g->nz + 1);
    size_t off = 0;
    auto take = [&](size_t bytes) -> char * {
        off = (off + 255) & ~(size_t)255;
        char *p = base ? base + off : nullptr;
        off += bytes;
        return p;
    };
    B **bulk[] = {&w->ax, &w->ay, &w->delpc, &w->ptc, &w->wc, &w->ke, &w->ut, &w->vt, &w->crx, &w->cry,
                  &w->xfx, &w->yfx, &w->FX, &w->FY, &w->VX, &w->VY, &w->dn, &w->pn, &w->wn, &w->om, &w->qo};
    for (auto p : bulk) *p = (B *)take(el * sizeof(B));
    double **f64[] = {&w->s1, &w->s2, &w->dp1, &w->dp2, &w->mxs, &w->mys};
    for (auto p : f64) *p = (double *)take(el * sizeof(double));
    double **f64i[] = {&w->pkc, &w->gz, &w->zh, &w->zn};
    for (auto p : f64i) *p = (double *)take(ei * sizeof(double));
    w->umax = (unsigned long long *)take(64);
    w->part = (double *)take(2 * part_count(g) * sizeof(double));
    return off + 256;
}

// block partials of MNF fields, and their sums
long reduction_elems(const fv3_grid *g) { return 2 * part_count(g) * MNF + MNF; }

void timing_start(const char *filter)
{
    g_timing.on = filter != nullptr;
    g_timing.filter = filter ? filter : "";
    g_timing.recs.clear();
}

int timing_stop(char *names, int names_cap, double *total_ms, long *counts, int cap)
{
    g_timing.on = false;
    if (hipDeviceSynchronize() != hipSuccess) return (int)FV3_EDEVICE;
    std::vector<std::string> keys;
    std::vector<double> tot;
    std::vector<long> cnt;
    for (TimingRec &r : g_timing.recs) {
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, r.a, r.b);
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
        size_t q = 0;
        while (q < keys.size() && keys[q] != r.name) q++;
        if (q == keys.size()) {
            keys.push_back(r.name);
            tot.push_back(0.0);
            cnt.push_back(0);
        }
        tot[q] += ms;
        cnt[q] += 1;
    }
    g_timing.recs.clear();
    int nk = 0, pos = 0;
    for (size_t q = 0; q < keys.size() && nk < cap; q++) {
        int len = (int)keys[q].size() + 1;
        if (pos + len > names_cap) break;
        std::memcpy(names + pos, keys[q].c_str(), len);
        pos += len;
        total_ms[nk] = tot[q];
        counts[nk] = cnt[q];
        nk++;
    }
    return nk;
}

size_t workspace_bytes(const fv3_grid *g)
{
    if (g->bulk_bytes == 4) {
        Work<float> w;
        return carve(g, nullptr, &w);
    }
    Work<double> w;
    return carve(g, nullptr, &w);
}

template <class B>
static Mets<B> metrics_b(const fv3_grid *g);
template <>
Mets<double> metrics_b<double>(const fv3_grid *g)
{
    Mets<double> M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = g->met[m];
    return M;
}
template <>
Mets<float> metrics_b<float>(const fv3_grid *g)
{
    Mets<float> M;
    for (int m = 0; m < M_ALL; m++) M.m[m] = g->metf[m];
    return M;
}
static MetD metrics_d(const fv3_grid *g) { return metrics_b<double>(g); }

// ====================================================================
// Host orchestration of one call
// ====================================================================
template <class B>
static fv3_status substeps_t(fv3_state *s, const fv3_grid *g, double dt, int n_split, int stop_stage,
                             hipStream_t st)
{
    Work<B> W;
    carve(g, (char *)s->workspace, &W);
    Mets<B> M = metrics_b<B>(g);
    MetD Md = metrics_d(g);
    const Geo &G = g->geo;
    int n = g->n, nz = g->nz, T = g->T, P = T * nz;
    long el = alloc_elems(g, nz);
    B *u = (B *)s->u, *v = (B *)s->v, *w = (B *)s->w, *delp = (B *)s->delp, *pt = (B *)s->pt;
    B *uc = (B *)s->uc, *vc = (B *)s->vc, *cx = (B *)s->cx, *cy = (B *)s->cy;
    double *delz = s->delz;
    const double *phis = s->phis;
    double bdt = dt / n_split, dt2 = 0.5 * bdt;
    const B *areaB = M.m[M_AREA];
    const B *qvp = (const B *)s->qv;
    const bool efix = g->p.edge_fix && g->edge_count > 0;

    // humidity is constant over the call: its halo once
    if (qvp) halo_set<B>(g, FieldSet<B>{{(B *)s->qv, nullptr, nullptr, nullptr}}, 1, nz, st);
    fill(s->mfx, el, 0.0, st);
    fill(s->mfy, el, 0.0, st);
    fill(cx, el, (B)0, st);
    fill(cy, el, (B)0, st);
    copy(delp, s->dp0, el, st);
    // interface heights: from the thicknesses once, then by every substep's
    // second column solve
    double *zI = W.zh;
    column_heights(g, delz, phis, zI, st);
    rec_mark();

    for (int it = 0; it < n_split; it++) {
        bool last = it == n_split - 1;
#define STOP(x) if (last && stop_stage == (x)) goto done
        // H-A
        halo_pair(g, g->planD, u, v, nz, st);
        halo_set<B>(g, FieldSet<B>{{delp, pt, w, nullptr}}, 3, nz, st);
        if (g->planC.count > 0)
            launch_fn<k_halo_z>("k_halo_z", dim3((g->planC.count + 255) / 256, nz + 1), dim3(256), st, G,
                                (const HaloEnt *)g->planC.d, g->planC.count, phis, zI, nz + 1, last ? delz : (double *)nullptr);
        STOP(1);
        // c_sw
        {
            CswArgs<B> a{};
            a.dt2 = (B)dt2;
            a.u = u; a.v = v; a.delp = delp; a.pt = pt; a.w = w;
            a.uc = uc; a.vc = vc; a.delpc = W.delpc; a.ptc = W.ptc; a.wc = W.wc; a.ax = W.ax; a.ay = W.ay;
            csw(g, a, st);
        }
        STOP(2);
        // dz_c + riem_solver_c on the half-step cells
        {
            ColArgs<B> a{};
            a.dt = dt2; a.beta = g->p.beta; a.ptop = g->p.ptop; a.cubic = g->p.pp_order == 4;
            a.dpi = W.delpc; a.theta = W.ptc; a.w = W.wc; a.qv = qvp; a.phis = phis;
            a.z = zI; a.ax = W.ax; a.ay = W.ay; a.pfull = W.pkc; a.phi = W.gz;
            column_solve<B, 0>(g, a, st);
        }
        STOP(3);
        launch2d_s(k_pgradc<B>, (Shape{32, 8}), 0, n, 0, n, T * ((nz + PGK - 1) / PGK), st, G, Md, dt2, (const B *)W.delpc, (const double *)W.pkc,
                 (const double *)W.gz, uc, vc);
        STOP(4);
        halo_pair(g, g->planCv, uc, vc, nz, st);
        STOP(5);
        // d_sw
        {
            // four layers a thread where that leaves four wavefronts on every SIMD
            const int layers = (long)(n + 6) * (n + 6) * P / 64 >= 4 * 4096 ? 4 : 1;
            launch2d_s(k_dsw_courant<B>, (sizeof(B) == 4 ? Shape{32, 8} : Shape{16, 16}), -3, n + 2, -3, n + 2,
                       T * ((nz + layers - 1) / layers), st, G, M, layers, (B)bdt, (const B *)uc, (const B *)vc, W.ut,
                       W.vt, W.crx, W.cry, W.xfx, W.yfx, g->flags);
        }
        const bool eppm = g->p.edge_ppm && g->p.kind == FV3_GRID_CUBED_SPHERE;
        // the marching transports' common arguments
        MarchArgs<B> ma{};
        ma.crx = W.crx; ma.cry = W.cry; ma.xfx = W.xfx; ma.yfx = W.yfx; ma.area = areaB;
        if (!eppm) {
            MarchArgs<B> a = ma;
            a.q[0] = delp; a.q[1] = pt; a.q[2] = w;
            a.out[0] = W.dn; a.out[1] = W.pn; a.out[2] = W.wn;
            a.mfx = s->mfx; a.mfy = s->mfy; a.cxa = cx; a.cya = cy;
            // edge-flux fix-up: keep the tile-edge fluxes (the C-grid half-step
            // arrays are free after p_grad_c)
            if (efix) {
                a.FX[0] = W.FX; a.FX[1] = W.delpc; a.FX[2] = W.wc;
                a.FY[0] = W.FY; a.FY[1] = W.ptc; a.FY[2] = W.qo;
            }
            march_mass(g, a, st);
        } else {
            FvArgs<B, B, B> a{};
            a.q = delp; a.Lq = nz; a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx;
            a.Lc = nz; a.area = areaB; a.epi = EPI_DELP; a.FX = W.FX; a.FY = W.FY; a.qout = W.dn;
            a.mfx = s->mfx; a.mfy = s->mfy; a.cxa = cx; a.cya = cy;
            fvtp(g, P, a, st);
            FvArgs<B, B, B> b{};
            b.q = pt; b.Lq = nz; b.crx = W.crx; b.cry = W.cry; b.xfx = W.xfx; b.yfx = W.yfx; b.Lc = nz;
            b.mx = W.FX; b.my = W.FY; b.area = areaB; b.epi = EPI_MASSW; b.qout = W.pn; b.dold = delp; b.dnew = W.dn;
            // edge-flux fix-up: keep the content fluxes (the C-grid half-step
            // arrays are free after p_grad_c)
            if (efix) { b.FX = W.delpc; b.FY = W.ptc; b.edges_only = 1; }
            fvtp(g, P, b, st);
            b.q = w; b.qout = W.wn;
            if (efix) { b.FX = W.wc; b.FY = W.qo; }
            fvtp(g, P, b, st);
        }
        // higher-order divergence damping (nord 1, 2): the C-grid half-step
        // arrays ax, ay are free after p_grad_c and hold the corner fields
        const B *hd = nullptr;
        double hc = 0.0;
        if (g->p.nord > 0 && g->p.d4_bg > 0.0) {
            launch2d(k_cdiv<B>, 0, n, 0, n, P, st, G, M, (const B *)u, (const B *)v, W.ax);
            B *a = W.ax, *b = W.ay;
            for (int r = 0; r < g->p.nord; r++) {
                halo_corner(g, a, nz, st);
                launch2d(k_clap<B>, 0, n, 0, n, P, st, G, M, (const B *)a, b);
                std::swap(a, b);
            }
            hd = a;
            hc = (g->p.nord % 2 ? 1.0 : -1.0) * std::pow(g->p.d4_bg * g->da_min, g->p.nord + 1);
        }
        auto omke = [&](auto lim) {
            if constexpr (sizeof(B) == 4)
                launch_fn<k_dsw_omke<B, decltype(lim)::value>>(
                    "k_dsw_omke<B>", dim3((unsigned)(((n + 6) * (n + 6) + 255) / 256), 1, (unsigned)P), dim3(256), st,
                    0, -3, n + 2, -3, n + 2, G, M, (B)bdt, (B)g->p.d2_bg, (B)(g->p.dddmp * bdt), (B)g->da_min,
                    (const B *)u, (const B *)v, (const B *)W.ut, (const B *)W.vt, (const B *)hd, (B)hc, W.om, W.ke);
            else
                launch2d_sh<k_dsw_omke<B, decltype(lim)::value>>(
                    "k_dsw_omke<B>", Shape{16, 16}, -3, n + 2, -3, n + 2, P, st, G, M, (B)bdt, (B)g->p.d2_bg,
                    (B)(g->p.dddmp * bdt), (B)g->da_min, (const B *)u, (const B *)v, (const B *)W.ut,
                    (const B *)W.vt, (const B *)hd, (B)hc, W.om, W.ke);
        };
        if (g->p.hord == 6) omke(std::integral_constant<int, 6>{});
        else if (g->p.hord == 5) omke(std::integral_constant<int, 5>{});
        else omke(std::integral_constant<int, 8>{});
        if (eppm) {
            const int cnt = 12 * (n + 1) - 36;
            auto kee = [&](auto lim) {
                launch_fn<k_ke_edge<B, decltype(lim)::value>>("k_ke_edge", dim3((cnt + 255) / 256, nz, 6), dim3(256),
                                                             st, G, M, (B)bdt, (const B *)u, (const B *)v,
                                                             (const B *)W.ut, (const B *)W.vt, W.ke);
            };
            if (g->p.hord == 6) kee(std::integral_constant<int, 6>{});
            else if (g->p.hord == 5) kee(std::integral_constant<int, 5>{});
            else kee(std::integral_constant<int, 8>{});
        }
        if (!eppm) {
            MarchArgs<B> a = ma;
            a.q[0] = W.om;
            a.ke = W.ke; a.u = u; a.v = v;
            a.rdx = M.m[M_RDX]; a.rdy = M.m[M_RDY]; a.rdxc = M.m[M_RDXC]; a.rdyc = M.m[M_RDYC]; a.fc = M.m[M_FC];
            a.nuv = (B)(g->p.vtdm * g->da_min);
            march_wind(g, a, st);
        } else {
            FvArgs<B, B, B> a{};
            a.q = W.om; a.Lq = nz; a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx; a.Lc = nz;
            a.area = areaB; a.epi = EPI_FLUX; a.FX = W.VX; a.FY = W.VY;
            fvtp(g, P, a, st);
            launch2d_s(k_dsw_update<B>, (Shape{32, 8}), 0, n, 0, n, P, st, G, M, (const B *)W.ke, (const B *)W.VX, (const B *)W.VY,
                 (const B *)W.om, (B)(g->p.vtdm * g->da_min), u, v);
        }
        if (efix)
            launch_fn<k_edgefix_dsw<B>>("k_edgefix", dim3((g->edge_count + 255) / 256, nz), dim3(256), st, G,
                                        (const EdgeCell *)g->edge_cells, g->edge_count, areaB, (const B *)W.FX,
                                        (const B *)W.FY, (const B *)W.delpc, (const B *)W.ptc, (const B *)W.wc,
                                        (const B *)W.qo, W.dn, W.pn, W.wn, s->mfx, s->mfy);
        if (last && (stop_stage == 6 || stop_stage == 7))
            launch2d(k_commit<B>, 0, n - 1, 0, n - 1, P, st, G, (const B *)W.dn, (const B *)W.pn, (const B *)W.wn, delp,
                     pt, w);
        STOP(6);
        // dz_d
        // (mixed: the deviations and their references in the scratch columns)
        double *zref = W.s2;
        if (!eppm) {
            MarchArgs<B> a = ma;
            a.z = zI; a.zref = zref; a.out[0] = (B *)W.zn;
            march_height(g, a, st);
        } else if constexpr (std::is_same<B, float>::value) {
            float *zd = (float *)W.s1;
            launch2d(k_zdev, -3, n + 2, -3, n + 2, g->T * (nz + 1), st, G, (const double *)zI, zref, zd);
            FvArgs<float, B, double> a{};
            a.q = zd; a.Lq = nz + 1; a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx; a.Lc = nz;
            a.iface = 1; a.area = M.m[M_AREA]; a.epi = EPI_ADV; a.qout = (float *)W.zn;
            fvtp(g, P, a, st);
        } else {
            FvArgs<double, B, double> a{};
            a.q = zI; a.Lq = nz + 1; a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx; a.Lc = nz;
            a.iface = 1; a.area = Md.m[M_AREA]; a.epi = EPI_ADV; a.qout = W.zn;
            fvtp(g, P, a, st);
        }
        if (last && stop_stage == 7) {
            if constexpr (std::is_same<B, float>::value)
                launch2d(k_delz_from_zdev, 0, n - 1, 0, n - 1, P, st, G, (const float *)W.zn, (const double *)zref,
                         phis, delz);
            else
                launch2d(k_delz_from_zh, 0, n - 1, 0, n - 1, P, st, G, (const double *)W.zn, phis, delz);
        }
        STOP(7);
        // riem_solver3; commits delp, pt, w, delz
        {
            ColArgs<B> a{};
            a.dt = bdt; a.beta = g->p.beta; a.ptop = g->p.ptop; a.cubic = g->p.pp_order == 4;
            a.dpi = W.dn; a.theta = W.pn; a.w = W.wn; a.qv = qvp; a.phis = phis;
            a.zt = W.zn; a.zref = zref; a.pfull = s->pfull; a.phi = s->phi;
            a.w_out = w; a.delp_out = delp; a.pt_out = pt; a.delz_out = delz; a.z_out = zI;
            column_solve<B, 1>(g, a, st);
        }
        STOP(8);
        // H-C
        halo_set<double>(g, FieldSet<double>{{s->pfull, s->phi, nullptr, nullptr}}, 2, nz + 1, st);
        halo_scalar(g, delp, nz, st);
        STOP(9);
        // nh_p_grad
        {
            NhArgs<B> a{};
            a.bdt = bdt; a.pfull = s->pfull; a.phi = s->phi; a.delp = delp; a.u = u; a.v = v;
            nh_grad(g, a, st);
        }
#undef STOP
    }
    rec_mark();
done:
    {
        B *chk[] = {u, v, w, delp, pt};
        for (B *f : chk) launch2d(k_check_finite<B>, 0, n - 1, 0, n - 1, P, st, G, nz, (const B *)f, g->flags);
        launch2d(k_check_finite<double>, 0, n - 1, 0, n - 1, P, st, G, nz, (const double *)delz, g->flags);
    }
    if (hipGetLastError() != hipSuccess) return FV3_EDEVICE;
    return FV3_OK;
}

fv3_status record_substeps(fv3_state *s, const fv3_grid *g, double bdt, Recorder *rec)
{
    rec->pos = 0;
    rec->mark = 0;
    g_rec = rec;
    fv3_status r = g->bulk_bytes == 4 ? substeps_t<float>(s, g, bdt, 1, 0, nullptr)
                                      : substeps_t<double>(s, g, bdt, 1, 0, nullptr);
    g_rec = nullptr;
    if (r != FV3_OK) return r;
    // a member whose options choose other kernels than the first member's
    if (rec->bad || rec->pos != rec->sites.size() || rec->mark != 2) return FV3_EUNSUPPORTED;
    return FV3_OK;
}

fv3_status run_substeps(fv3_state *s, const fv3_grid *g, double dt, int n_split, int stop_stage,
                        hipStream_t st)
{
    if (g->bulk_bytes == 4) return substeps_t<float>(s, g, dt, n_split, stop_stage, st);
    return substeps_t<double>(s, g, dt, n_split, stop_stage, st);
}

fv3_status run_halo_cells(const fv3_grid *g, void *const *f, int nf, int levels, int fp64,
                          hipStream_t st)
{
    for (int q = 0; q < nf; q++) {
        if (fp64 || g->bulk_bytes == 8) halo_scalar(g, (double *)f[q], levels, st);
        else halo_scalar(g, (float *)f[q], levels, st);
    }
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

fv3_status run_halo_pair_cells(const fv3_grid *g, void *fx, void *fy, int levels, int fp64,
                               hipStream_t st)
{
    if (fp64 || g->bulk_bytes == 8) halo_pair(g, g->planA, (double *)fx, (double *)fy, levels, st);
    else halo_pair(g, g->planA, (float *)fx, (float *)fy, levels, st);
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

template <class B>
static fv3_status tracer_t(void *const *q, int nq, fv3_state *s, const fv3_grid *g, int nsplt, hipStream_t st)
{
    Work<B> W;
    carve(g, (char *)s->workspace, &W);
    Mets<B> M = metrics_b<B>(g);
    MetD Md = metrics_d(g);
    const Geo &G = g->geo;
    int n = g->n, nz = g->nz, P = g->T * nz;
    long el = alloc_elems(g, nz);
    B *cx = (B *)s->cx, *cy = (B *)s->cy;
    halo_pair(g, g->planCv, cx, cy, nz, st);
    if (nsplt <= 0) {
        unsigned long long zero = 0, h = 0;
        fill(W.umax, 1, zero, st);
        launch2d_native("k_absmax", k_absmax<B>, 0, n, 0, n, P < 8 ? P : 8, st, G, (const B *)cx, (const B *)cy,
                        W.umax);
        if (hipMemcpyAsync(&h, W.umax, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess) return FV3_EDEVICE;
        if (hipStreamSynchronize(st) != hipSuccess) return FV3_EDEVICE;
        double cmax;
        std::memcpy(&cmax, &h, sizeof(cmax));
        if (!std::isfinite(cmax))
            return set_error(FV3_ENONFINITE, "accumulated Courant numbers cx, cy are not finite");
        if (cmax > (double)FV3_MAX_TRACER_SUBCYCLES)
            return set_error(FV3_ECFL, "max |cx|, |cy| = " + std::to_string(cmax) + " needs more than " +
                                           std::to_string(FV3_MAX_TRACER_SUBCYCLES) + " tracer sub-cycles");
        nsplt = (int)std::ceil(cmax);
        if (nsplt < 1) nsplt = 1;
    }
    double rs = (double)nsplt;
    const bool efix = g->p.edge_fix && g->edge_count > 0;
    const bool eppm = g->p.edge_ppm && g->p.kind == FV3_GRID_CUBED_SPHERE;
    launch2d_s(k_tracer_flux<B>, (Shape{128, 2}), -3, n + 3, -3, n + 3, P, st, G, Md, rs, (const B *)cx, (const B *)cy,
             (const double *)s->mfx, (const double *)s->mfy, W.crx, W.cry, W.xfx, W.yfx, eppm ? W.mxs : (double *)nullptr,
             eppm ? W.mys : (double *)nullptr);
    if (!eppm) {
        // up to MARCH_TRACERS fields at a time, each sub-cycle from the fields to
        // scratch or back
        B *scr[MARCH_TRACERS] = {W.qo, W.dn, W.pn, W.wn};
        B *efx[MARCH_TRACERS] = {W.delpc, W.wc, W.ut, W.VX}, *efy[MARCH_TRACERS] = {W.ptc, W.ke, W.vt, W.VY};
        MarchArgs<B> a{};
        a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx; a.area = M.m[M_AREA];
        a.mx = s->mfx; a.my = s->mfy; a.area64 = Md.m[M_AREA]; a.rs = rs;
        struct Group {
            FieldSet<B> src, dst;
            int nf;
        } gs[64];   // as many as there are tracers, at most
        int ng = 0;
        bool repeated = false;
        for (int m = 0; m < nq; m++) {
            for (int f = 0; f < m; f++) repeated |= q[f] == q[m];
            // a field given twice is transported twice, one after the other
            bool again = false;
            if (ng > 0)
                for (int f = 0; f < gs[ng - 1].nf; f++) again |= gs[ng - 1].src.p[f] == (B *)q[m];
            if (ng == 0 || again || gs[ng - 1].nf == (sizeof(B) == 4 ? MARCH_TRACERS : 3)) gs[ng++] = Group{};
            Group &t = gs[ng - 1];
            t.src.p[t.nf] = (B *)q[m];
            t.dst.p[t.nf] = scr[t.nf];
            t.nf++;
        }
        auto subcycle = [&](Group &t, int itr) {
            halo_set<B>(g, t.src, t.nf, nz, st);
            for (int f = 0; f < t.nf; f++) {
                a.q[f] = t.src.p[f];
                a.out[f] = t.dst.p[f];
                a.FX[f] = efix ? efx[f] : nullptr;
                a.FY[f] = efix ? efy[f] : nullptr;
            }
            a.dp1 = itr == 0 ? s->dp0 : itr % 2 ? W.dp1 : W.dp2;
            a.dp2 = itr + 1 < nsplt || efix ? (itr % 2 ? W.dp2 : W.dp1) : nullptr;
            march_tracer(g, t.nf, a, st);
            if (efix)
                for (int f = 0; f < t.nf; f++)
                    launch_fn<k_edgefix_q<B>>("k_edgefix_q", dim3((g->edge_count + 255) / 256, nz), dim3(256), st, G,
                                              (const EdgeCell *)g->edge_cells, g->edge_count,
                                              (const B *)M.m[M_AREA], (const B *)a.FX[f], (const B *)a.FY[f],
                                              (const double *)a.dp2, t.dst.p[f]);
            std::swap(t.src, t.dst);
        };
        auto back = [&](Group &t) {   // from scratch into the fields
            launch2d_s(k_copy_back<B>, (Shape{128, 2}), 0, n - 1, 0, n - 1, P * t.nf, st, G, P, t.src, t.dst);
            std::swap(t.src, t.dst);
        };
        if (!repeated) {
            for (int k = 0; k < ng; k++) {
                for (int itr = 0; itr < nsplt; itr++) subcycle(gs[k], itr);
                if (nsplt % 2) back(gs[k]);
                halo_set<B>(g, gs[k].src, gs[k].nf, nz, st);   // leave consistent halos
            }
        } else {
            // every sub-cycle of a repeated field follows all of the one before
            for (int itr = 0; itr < nsplt; itr++)
                for (int k = 0; k < ng; k++) {
                    subcycle(gs[k], itr);
                    back(gs[k]);
                }
            for (int k = 0; k < ng; k++) halo_set<B>(g, gs[k].src, gs[k].nf, nz, st);
        }
        return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
    }
    copy(s->dp0, W.dp1, el, st);
    double *dp1 = W.dp1, *dp2 = W.dp2;
    for (int itr = 0; itr < nsplt; itr++) {
        launch2d(k_tracer_dp, 0, n - 1, 0, n - 1, P, st, G, Md, (const double *)dp1, (const double *)W.mxs,
                 (const double *)W.mys, dp2);
        for (int m = 0; m < nq; m++) {
            B *Q = (B *)q[m];
            halo_scalar(g, Q, nz, st);
            FvArgs<B, B, double> a{};
            a.q = Q; a.Lq = nz; a.crx = W.crx; a.cry = W.cry; a.xfx = W.xfx; a.yfx = W.yfx; a.Lc = nz;
            a.mx = W.mxs; a.my = W.mys; a.area = M.m[M_AREA]; a.epi = EPI_TRACER; a.qout = W.qo;
            a.dp1 = dp1; a.dp2 = dp2;
            if (efix) { a.FX = W.delpc; a.FY = W.ptc; a.edges_only = 1; }
            fvtp(g, P, a, st);
            copy((const B *)W.qo, Q, el, st);
            if (efix)
                launch_fn<k_edgefix_q<B>>("k_edgefix_q", dim3((g->edge_count + 255) / 256, nz), dim3(256), st, G,
                                          (const EdgeCell *)g->edge_cells, g->edge_count, (const B *)M.m[M_AREA],
                                          (const B *)W.delpc, (const B *)W.ptc, (const double *)dp2, Q);
        }
        double *tmp = dp1;
        dp1 = dp2;
        dp2 = tmp;
    }
    for (int m = 0; m < nq; m++) halo_scalar(g, (B *)q[m], nz, st);   // leave consistent halos
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

fv3_status run_tracer(void *const *q, int nq, fv3_state *s, const fv3_grid *g, int nsplt,
                      hipStream_t st)
{
    if (g->bulk_bytes == 4) return tracer_t<float>(q, nq, s, g, nsplt, st);
    return tracer_t<double>(q, nq, s, g, nsplt, st);
}

// block partials of fields w0 .. w0 + nf - 1 (0: mass, 1: pt, 2 + m: q[m])
template <class B>
static void mass_partials(const fv3_grid *g, const void *delp, const void *pt, void *const *q, int w0, int nf, double *part,
                          hipStream_t st)
{
    MassFields<B> F{};
    F.nf = nf;
    for (int f = 0; f < nf; f++) F.p[f] = (const B *)(w0 + f == 0 ? nullptr : w0 + f == 1 ? pt : q[w0 + f - 2]);
    launch2d_native("k_mass_partial", k_mass_partial<B>, 0, g->n - 1, 0, g->n - 1, g->T, st, g->geo, metrics_d(g),
                    (const B *)delp, F, part);
}
static void mass_final(const fv3_grid *g, int nf, const double *part, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_mass_final, dim3((unsigned)nf), dim3(256), 0, st, part, part_count(g), out);
}

// k_mass_final's combination on the host
static double mass_combine(const double *part, long np)
{
    double s = 0.0, c = 0.0;
    for (long b = 0; b < np; b++) {
        const double x = part[2 * b], t = s + x;
        const bool big = std::fabs(s) >= std::fabs(x);
        c = (c + part[2 * b + 1]) + (((big ? s : x) - t) + (big ? x : s));
        s = t;
    }
    return s + c;
}

template <class B>
static fv3_status mass_sums_t(const fv3_grid *g, const void *delp, const void *pt, void *const *q,
                              int nq, double *out, hipStream_t st)
{
    const long np = part_count(g);
    double *dout = g->red + 2 * np * MNF;
    for (int w0 = 0; w0 < 2 + nq; w0 += MNF) {
        const int nf = 2 + nq - w0 < MNF ? 2 + nq - w0 : MNF;
        mass_partials<B>(g, delp, pt, q, w0, nf, g->red, st);
        // A host thread makes the same additions in the same order in a quarter
        // of the time of one of the device, but after a copy of all partials,
        // whose first call costs about 100 us more.  It is taken for few fields of
        // many blocks (two sums, device / host: 1024 x 1024 x 2 110 / 63 us, C384 x
        // 20 121 / 80, C768 x 3 259 / 130); six sums are 115 / 104, 149 / 137 and
        // 281 / 282, those of C192 x 79 126 / 120 (first call 212 / 320 to 430).
        if (nf <= 3 && np >= 2048) {
            std::vector<double> h((size_t)(2 * np * nf));
            if (hipMemcpyAsync(h.data(), g->red, h.size() * sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess)
                return FV3_EDEVICE;
            for (int f = 0; f < nf; f++) out[w0 + f] = mass_combine(&h[(size_t)(2 * np * f)], np);
            continue;
        }
        mass_final(g, nf, g->red, dout, st);
        if (hipMemcpyAsync(out + w0, dout, nf * sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess)
            return FV3_EDEVICE;
        if (hipStreamSynchronize(st) != hipSuccess) return FV3_EDEVICE;
    }
    return FV3_OK;
}

// Streaming copy for the bandwidth roof: 16-byte loads and stores; a block
// moves 16 KiB per iteration (four loads per thread issued before the four
// stores), grid-stride over 16 KiB chunks with at most 2048 blocks (8 per
// compute unit).
__global__ void __launch_bounds__(256) k_stream_copy(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                     long n16)
{
    const long stride = (long)gridDim.x * 1024;
    for (long base = (long)blockIdx.x * 1024; base < n16; base += stride) {
        uint4 r[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            long e = base + u * 256 + threadIdx.x;
            if (e < n16) r[u] = src[e];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            long e = base + u * 256 + threadIdx.x;
            if (e < n16) dst[e] = r[u];
        }
    }
}

fv3_status run_device_copy(const void *src, void *dst, size_t bytes, hipStream_t st)
{
    long n16 = (long)(bytes / 16);
    bool tm = timing_wanted("k_stream_copy");
    TimingRec r;
    if (tm) timing_begin("k_stream_copy", st, r);
    if (n16 > 0) {
        long chunks = (n16 + 1023) / 1024;
        unsigned blocks = (unsigned)(chunks < 2048 ? chunks : 2048);
        hipLaunchKernelGGL(k_stream_copy, dim3(blocks), dim3(256), 0, st, (const uint4 *)src, (uint4 *)dst, n16);
    }
    if (tm) timing_end(st, r);
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

fv3_status run_mass_sums(const fv3_grid *g, const void *delp, const void *pt, void *const *q,
                         int nq, double *out, hipStream_t st)
{
    if (g->bulk_bytes == 4) return mass_sums_t<float>(g, delp, pt, q, nq, out, st);
    return mass_sums_t<double>(g, delp, pt, q, nq, out, st);
}

// ====================================================================
// Allocation-free mass sums.  The per-block partials go to a fixed
// file-scope device array instead of the grid's reduction buffer, and one
// thread combines them on the device into the caller's device output, so
// the call allocates nothing (device or host) and does not synchronise.
// Each GPU holds its own copy of the array; host code only ever uses the
// address that hipGetSymbolAddress returned for the current device.
// ====================================================================
static __device__ __align__(256) double scratch[FV3_NOALLOC_SCRATCH_BYTES / sizeof(double)];

static std::mutex g_scratch_mu;
static double *g_scratch_dev[FV3_MAX_DEVICES];   // device address of `scratch`, per HIP ordinal

fv3_status noalloc_setup(int device)
{
    if (device < 0 || device >= FV3_MAX_DEVICES) return FV3_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_dev[device]) return FV3_OK;
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FV3_EDEVICE;
    g_scratch_dev[device] = (double *)p;
    return FV3_OK;
}

long noalloc_mass_doubles(const fv3_grid *g) { return 2 * part_count(g); }

template <class B>
static fv3_status mass_sums_noalloc_t(const fv3_grid *g, const void *delp, const void *pt, void *const *q,
                                      int nq, double *dev_out, double *part, hipStream_t st)
{
    // as many fields a pass as the scratch holds; every block of
    // k_mass_partial writes its own slots (zero outside the interior), so
    // nothing in the scratch has to be cleared first
    const long cap = (long)(FV3_NOALLOC_SCRATCH_BYTES / sizeof(double)) / noalloc_mass_doubles(g);
    const int most = cap < MNF ? (int)cap : MNF;
    for (int w0 = 0; w0 < 2 + nq; w0 += most) {
        const int nf = 2 + nq - w0 < most ? 2 + nq - w0 : most;
        mass_partials<B>(g, delp, pt, q, w0, nf, part, st);
        mass_final(g, nf, part, dev_out + w0, st);
    }
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

fv3_status run_mass_sums_noalloc(const fv3_grid *g, const void *delp, const void *pt, void *const *q,
                                 int nq, double *dev_out, hipStream_t st)
{
    double *part = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (g->p.device >= 0 && g->p.device < FV3_MAX_DEVICES) part = g_scratch_dev[g->p.device];
    }
    if (!part) return FV3_EINTERNAL;   // fv3_init_grid resolves it for the grid's device
    if (g->bulk_bytes == 4) return mass_sums_noalloc_t<float>(g, delp, pt, q, nq, dev_out, part, st);
    return mass_sums_noalloc_t<double>(g, delp, pt, q, nq, dev_out, part, st);
}

}  // namespace fv3
