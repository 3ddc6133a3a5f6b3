// Vertical remapping of the remapping step (Sec. II): the deformed Lagrangian
// layers of every column are mapped back to the reference interfaces
// pe_K = ak_K + bk_K ps (ps = ptop + the column's sum of delp) by a
// mass-conserving piecewise-parabolic remap in pressure.
//
// Reconstruction (Colella-Woodward PPM on non-uniform layers): interface
// values by fourth-order interpolation of the layer means with monotonised
// slopes where two layers lie on each side, thickness-weighted linear
// interpolation next to the top and bottom layers, constant top and bottom
// layers, and the monotonicity limiter on each parabola.  Fields: pt, w and
// the tracers as they are, delz as delz/delp (its remapped integral is the
// new delz, so the column depth is kept), the D-grid winds at faces on the
// mean interfaces of the two cells that share the face; delp becomes the
// reference thickness.
//
// GPU mapping: a block's 256 threads take 16 to 256 columns and cut them into
// 16 to 1 chunks of target layers, one thread per (column, chunk).  The block
// sums the columns' interface pressures into LDS (in layer order) and stages
// the source columns of up to RNF fields there; then every thread finds the
// source layer that its first target layer starts in by bisection, rebuilds the
// interpolation state from the two layers above and walks on: per source layer
// it finishes the target layers that end in it, so that the threads of a
// wavefront advance together.  A window of means and thicknesses and the
// interface value below the current layer (which becomes the one above the
// next) stay in registers.  As every read of the walk is from LDS, results go
// straight into the fields.  All arithmetic is FP64; no value depends on the
// split.
//
// What bounds it is the instructions of the walk: some 240 a source layer and
// 50 more a field, with about ten divisions in a serial chain, and two or
// three layers per chunk to rebuild the state.  Measured, cells (seven fields)
// / both winds / whole remap: C48 x 79 mixed 496 / 534 / 1030 us as one thread
// per column with results in a workspace and copied back, 87 / 52 / 148 now;
// C192 x 79, eight fields, 3.78 -> 1.98 ms (FP64 4.14 -> 2.00).  On the way:
// 16 chunks without the staging, 8 chunks of 32 columns, 120 us for the cells
// (their loads wait for the stores before them); staged, 8 chunks of 32
// columns, 108 us with four fields a thread, 124 with three, 134 with two.
#include <algorithm>
#include <cmath>
#include <string>

#include "flog.hpp"
#include "fv3_internal.hpp"

namespace fv3 {
namespace {

constexpr int RMAX = FV3_REMAP_MAX_LEVELS;
constexpr int RFIELDS = 8;   // fields per launch, at most
constexpr int RNF = 4;      // cell fields per thread (one walk of the column serves them all)
constexpr int RNT = 256;    // threads per block: columns x chunks of layers
constexpr int RB = 8;       // loads of a thread in flight while it fills LDS
enum { RM_CELL = 0, RM_WIND = 1 };

// reference coordinate, passed by value in the kernel arguments
struct RCoef {
    double ak[RMAX + 1], bk[RMAX + 1];
};

struct RBatch {
    void *fld[RFIELDS];   // remapped in place
    int fp64[RFIELDS];    // 1: the field is FP64, else bulk precision
    int ratio[RFIELDS];   // 1: remap field / delp, store its integral (delz)
    int nf;
};

// element of a field of bulk type B, or of an FP64 one
template <class B>
__device__ __forceinline__ void st(void *p, long e, bool fp64, double v)
{
    if (fp64 || sizeof(B) == 8) ((double *)p)[e] = v;
    else ((float *)p)[e] = (float)v;
}
// monotonised slope from the raw slope and the two one-sided differences
__device__ __forceinline__ double mono(double raw, double lo, double hi)
{
    if (lo * hi <= 0.0) return 0.0;
    return copysign(fmin(fabs(raw), 2.0 * fmin(fabs(lo), fabs(hi))), raw);
}

// Split of a block: CW = 2^lw columns, thread (c, ch) works on chunk ch of
// column c; chunks of cs layers.
struct Split {
    int cw, c, ch, cs;
    __device__ __forceinline__ Split(int lw, int nz)
        : cw(1 << lw), c((int)threadIdx.x & (cw - 1)), ch((int)threadIdx.x >> lw),
          cs((nz + (RNT >> lw) - 1) / (RNT >> lw)) {}
};

// interface pressures of the block's columns, summed in layer order:
// pe[k * cw + c], k = 0 .. nz
template <class H>
__device__ __forceinline__ void interfaces(double *pe, int nz, double ptop, const Split &S, bool in, H thick)
{
    const int k1 = min(nz, (S.ch + 1) * S.cs);
    for (int k0 = S.ch * S.cs; k0 < k1; k0 += RB) {
        double h[RB];
#pragma unroll
        for (int q = 0; q < RB; q++) h[q] = in && k0 + q < k1 ? thick(k0 + q) : 1.0;   // all loads in flight
#pragma unroll
        for (int q = 0; q < RB; q++)
            if (k0 + q < k1) pe[(k0 + q + 1) * S.cw + S.c] = h[q];
    }
    __syncthreads();
    if (S.ch == 0) {
        double p = ptop;
        pe[S.c] = p;
        for (int k = 1; k <= nz; k += 8) {
            double h[8];
#pragma unroll
            for (int q = 0; q < 8; q++) h[q] = pe[min(k + q, nz) * S.cw + S.c];
#pragma unroll
            for (int q = 0; q < 8; q++) {
                p += h[q];
                if (k + q <= nz) pe[(k + q) * S.cw + S.c] = p;
            }
        }
    }
    __syncthreads();
}

// the thread's layers of a column to LDS (divided by delp, if given)
template <class T, class B>
__device__ __forceinline__ void stage(T *to, const void *from, const B *delp, long c0, long lev, int nz, const Split &S)
{
    const int k1 = min(nz, (S.ch + 1) * S.cs);
    for (int k0 = S.ch * S.cs; k0 < k1; k0 += RB) {
        T v[RB];
        B h[RB];
#pragma unroll
        for (int q = 0; q < RB; q++) {
            const long e = c0 + (long)(k0 + q) * lev;
            v[q] = k0 + q < k1 ? ((const T *)from)[e] : (T)0;
            h[q] = delp && k0 + q < k1 ? delp[e] : (B)1;
        }
#pragma unroll
        for (int q = 0; q < RB; q++)
            if (k0 + q < k1) to[(k0 + q) * S.cw + S.c] = delp ? (T)(v[q] * fdiv(1.0, (double)h[q])) : v[q];
    }
}

// Remap up to NF fields of a chunk of target layers of one column, cells
// (fields f0 .. of the batch) or faces (field 0: west-east faces of u, field
// 1: v).  The layer geometry (reciprocals of the thickness sums of the
// interface interpolation) is computed once per source layer for all fields;
// the limited slope of layer s + 1, needed by the interface below layer s, is
// kept for the interface below layer s + 1.
template <class B, int MODE, int NF>
__global__ __launch_bounds__(256) void k_remap(Geo G, int lw, double ptop, RCoef C, RBatch F, const B *delp, int *flags)
{
    extern __shared__ double lds[];
    const int n = G.n, nz = G.nz;
    const Split S(lw, nz);
    const int c = S.c, CW = S.cw;
    // interface pressures, coefficients, source fields
    double *pe = lds, *ab = pe + (nz + 1) * CW, *fld = ab + 2 * (nz + 1);
    if ((int)threadIdx.x <= nz) {
        // the coefficients by lane from LDS: the kernel arguments lie in host
        // memory, and the walk would wait for one at every target layer
        ab[threadIdx.x] = C.ak[threadIdx.x];
        ab[nz + 1 + threadIdx.x] = C.bk[threadIdx.x];
    }
    const int groups = MODE == RM_WIND ? 2 : (F.nf + NF - 1) / NF;
    const int t = (int)blockIdx.y / groups, f0 = (int)blockIdx.y % groups * NF;
    const int nfg = MODE == RM_WIND ? 1 : min(NF, F.nf - f0);
    const bool vface = MODE == RM_WIND && f0 == 1;
    const int ni = vface ? n + 1 : n, nj = MODE == RM_WIND && !vface ? n + 1 : n;
    const int col = (int)blockIdx.x * CW + c, j = col / ni, i = col - j * ni;
    const bool in = j < nj;
    const long lev = G.lev;
    const long c0 = G.off0 + (long)t * nz * lev + (long)j * G.pitch + i;
    const long c1 = vface ? c0 - 1 : c0 - G.pitch;   // other cell of a face
    auto thick = [&](int k) -> double {
        const long o = (long)k * lev;
        if (MODE == RM_CELL) return (double)delp[c0 + o];
        return 0.5 * ((double)delp[c0 + o] + (double)delp[c1 + o]);
    };
    const int m0 = S.ch * S.cs, m1 = min(nz, m0 + S.cs);
    // the source columns: every read of the walk is then from LDS, and its
    // stores, straight into the fields, are never waited for
    double *src[NF];
    bool ratio[NF], f64[NF];
    {
        double *at = fld;
#pragma unroll
        for (int q = 0; q < NF; q++) {
            src[q] = at;
            ratio[q] = f64[q] = false;
            if (q >= nfg) continue;
            ratio[q] = F.ratio[f0 + q] != 0;
            f64[q] = sizeof(B) == 8 || F.fp64[f0 + q] != 0;
            at += (f64[q] ? nz : (nz + 1) / 2) * CW;
            if (!in) continue;
            if (ratio[q]) stage<double>(src[q], F.fld[f0 + q], delp, c0, lev, nz, S);
            else if (f64[q]) stage<double>(src[q], F.fld[f0 + q], (const B *)nullptr, c0, lev, nz, S);
            else stage<float>((float *)src[q], F.fld[f0 + q], (const B *)nullptr, c0, lev, nz, S);
        }
    }
    interfaces(pe, nz, ptop, S, in, thick);
    const double ps = pe[nz * CW + c];
    const bool mine = in && m0 < m1;
    auto target = [&](int K) -> double {   // both coordinates end on ps exactly
        return K == 0 ? ptop : K < nz ? ab[K] + ab[nz + 1 + K] * ps : ps;
    };
    bool bad = false;
    if (mine) {
        double top2 = target(m0), bot2 = target(m0 + 1), cur = top2;
        // first source layer that ends below the chunk's top
        int lo = 0, hi = nz - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (pe[(mid + 1) * CW + c] > top2) hi = mid;
            else lo = mid + 1;
        }
        // The state of the walk at layer s: means of layers s, s + 1, s + 2
        // (a2..a4), thicknesses of s - 1 .. s + 2 (d1..d4), the limited slope
        // of s + 1 (sl3), the interface value below s (eR).  It starts two
        // layers above the first one that is integrated (or at the top).
        int s = max(lo - 2, 0);
        double d1 = 1, d2 = 1, d3 = 1, d4 = 1;
        double a2[NF], a3[NF], a4[NF], sl3[NF], eR[NF], l[NF], r[NF], c6[NF], acc[NF];
        auto layer = [&](int k, double *a, double &d) {
            if (k >= nz) return;
            d = pe[(k + 1) * CW + c] - pe[k * CW + c];
#pragma unroll
            for (int q = 0; q < NF; q++) {
                a[q] = f64[q] ? src[q][k * CW + c] : (double)((const float *)src[q])[k * CW + c];
            }
        };
        // limited slope of layer s + 1
        auto slope3 = [&](bool have) {
            const double rr = fdiv(1.0, d2 + d3 + d4), kh = fdiv(d3 * rr * (2.0 * d2 + d3), d4 + d3),
                         kl = fdiv(d3 * rr * (d3 + 2.0 * d4), d2 + d3);
#pragma unroll
            for (int q = 0; q < NF; q++) {
                const double dl = a3[q] - a2[q], dh = a4[q] - a3[q];
                sl3[q] = have ? mono(kh * dh + kl * dl, dl, dh) : 0.0;
            }
        };
        // interface value below layer s (K = s + 1); sl2 = the limited slope of layer s
        auto below = [&](const double *sl2) {
            const int K = s + 1;
            const double s23 = d2 + d3, rs = fdiv(1.0, s23);
            if (K >= 2 && K <= nz - 2) {
                const double rsum = fdiv(1.0, d1 + d2 + d3 + d4), cj = d2 * rs;
                const double e1 = 2.0 * d2 + d3, e2 = 2.0 * d3 + d2;
                const double q1 = fdiv(d1 + d2, e1), q2 = fdiv(d4 + d3, e2);
                const double w = 2.0 * d3 * d2 * rs * (q1 - q2), g1 = d3 * q2, g2 = d2 * q1;
#pragma unroll
                for (int q = 0; q < NF; q++) {
                    const double jump = a3[q] - a2[q];
                    eR[q] = a2[q] + cj * jump + (w * jump - g2 * sl3[q] + g1 * sl2[q]) * rsum;
                }
            } else {
#pragma unroll
                for (int q = 0; q < NF; q++) eR[q] = (a2[q] * d3 + a3[q] * d2) * rs;
            }
        };
#pragma unroll
        for (int q = 0; q < NF; q++) a2[q] = a3[q] = a4[q] = acc[q] = 0.0;
        if (s > 0) d1 = pe[(s) * CW + c] - pe[(s - 1) * CW + c];
        layer(s, a2, d2);
        layer(s + 1, a3, d3);
        layer(s + 2, a4, d4);
        slope3(s + 2 <= nz - 1);
        {
            // used at the top layer only, which is constant
            const double rs = fdiv(1.0, d2 + d3);
#pragma unroll
            for (int q = 0; q < NF; q++) {
                eR[q] = nz > 1 ? (a2[q] * d3 + a3[q] * d2) * rs : a2[q];
                l[q] = r[q] = a2[q];
                c6[q] = 0.0;
            }
        }
        int m = m0;
        for (;;) {
            const double top1 = pe[(s) * CW + c], bot1 = pe[(s + 1) * CW + c];
            if (s >= lo) {
                const double rds = fdiv(1.0, bot1 - top1);
                // integral over [x1, x2] of l + x (r - l + c6 (1 - x)), times the thickness
                auto part = [&](double nxt) {
                    const double x1 = (cur - top1) * rds, x2 = (nxt - top1) * rds;
                    const double h = nxt - cur, sx = 0.5 * (x1 + x2), qx = (x1 * x1 + x1 * x2 + x2 * x2) * (1.0 / 3.0);
#pragma unroll
                    for (int q = 0; q < NF; q++) acc[q] += h * (l[q] + (r[q] - l[q] + c6[q]) * sx - c6[q] * qx);
                    cur = nxt;
                };
                while (bot2 <= bot1) {   // target layers that end in layer s
                    part(bot2);
                    const double dm = bot2 - top2, rdm = fdiv(1.0, dm);
                    bad |= !(dm > 0.0);
#pragma unroll
                    for (int q = 0; q < NF; q++) {
                        if (q < nfg)
                            st<B>(F.fld[f0 + q], c0 + (long)m * lev, f64[q], ratio[q] ? acc[q] : acc[q] * rdm);
                        acc[q] = 0.0;
                    }
                    top2 = bot2;
                    if (++m == m1) break;
                    bot2 = target(m + 1);
                }
                if (m == m1) break;
                if (s == nz - 1) {   // a target interface below the surface
                    bad = true;
                    break;
                }
                part(bot1);
            }
            // into source layer s + 1
            s++;
            double sl2[NF], eL[NF];
#pragma unroll
            for (int q = 0; q < NF; q++) {
                a2[q] = a3[q];
                a3[q] = a4[q];
                sl2[q] = sl3[q];
                eL[q] = eR[q];
            }
            d1 = d2; d2 = d3; d3 = d4;
            layer(s + 2, a4, d4);
            slope3(s + 2 <= nz - 1);
            if (s < nz - 1) below(sl2);
#pragma unroll
            for (int q = 0; q < NF; q++) {
                double lq = eL[q], rq = eR[q];
                const double aq = a2[q];
                if (s == nz - 1 || (rq - aq) * (aq - lq) <= 0.0) {
                    lq = rq = aq;
                } else {
                    const double dq = rq - lq, cc = 6.0 * (aq - 0.5 * (lq + rq));
                    if (dq * cc > dq * dq) lq = 3.0 * aq - 2.0 * rq;
                    else if (-dq * dq > dq * cc) rq = 3.0 * aq - 2.0 * lq;
                }
                l[q] = lq;
                r[q] = rq;
                c6[q] = 6.0 * (aq - 0.5 * (lq + rq));
            }
        }
    }
    if (bad) atomicOr(flags + 2, 1);
}

// delp of every column becomes the reference thickness
template <class B>
__global__ __launch_bounds__(256) void k_remap_delp(Geo G, int lw, double ptop, RCoef C, B *delp)
{
    extern __shared__ double pe[];
    __shared__ double ab[2][RMAX + 1];
    const int n = G.n, nz = G.nz;
    const Split S(lw, nz);
    const int c = S.c, CW = S.cw;
    if ((int)threadIdx.x <= nz) {
        ab[0][threadIdx.x] = C.ak[threadIdx.x];
        ab[1][threadIdx.x] = C.bk[threadIdx.x];
    }
    const int col = (int)blockIdx.x * CW + c, j = col / n, i = col - j * n;
    const bool in = j < n;
    const long c0 = G.off0 + (long)blockIdx.y * nz * G.lev + (long)j * G.pitch + i;
    interfaces(pe, nz, ptop, S, in, [&](int k) -> double { return (double)delp[c0 + (long)k * G.lev]; });
    if (!in) return;
    const double ps = pe[nz * CW + c];
    const int k0 = S.ch * S.cs, k1 = min(nz, k0 + S.cs);
    double top = k0 == 0 ? ptop : ab[0][min(k0, nz)] + ab[1][min(k0, nz)] * ps;
    for (int k = k0; k < k1; k++) {
        const double bot = ab[0][k + 1] + ab[1][k + 1] * ps;
        delp[c0 + (long)k * G.lev] = (B)(bot - top);
        top = bot;
    }
}

template <class K, class... A>
void timed(const char *name, K kern, size_t lds, dim3 grd, dim3 blk, hipStream_t s, A... args)
{
    TimingRec r;
    bool tm = timing_wanted(name);
    if (tm) timing_begin(name, s, r);
    hipLaunchKernelGGL(kern, grd, blk, lds, s, args...);
    if (tm) timing_end(s, r);
}

// log2 of the columns per block: chunks of about five layers (each rebuilds the
// state of the two layers above it, and the shorter they are the fewer columns
// share the block's serial sums), 16 chunks at most, and no fewer than 128
// blocks where 16 columns a block give as many.  Whole remap with four tracers,
// mixed, us, 16 chunks / this rule (one thread per column, before the chunks):
// 512 x 512 x 7 periodic 449 / 137 (198), C384 x 20 2439 / 1133 (1788), C96 x 5
// 107 / 43 (92), C192 x 40 928 / 648 (1118); the same split at C192 x 79 (1395)
// and C48 x 79 (131), where chunks of ten layers take 1579 and 151.
int remap_shift(int nz, long columns)
{
    int lw = 8;
    while (lw > 4 && (RNT >> lw) * 5 < nz) lw--;
    while (lw > 4 && (columns >> lw) < 128) lw--;
    return lw;
}

template <class T>
fv3_status remap(fv3_state *s, const fv3_grid *g, const double *ak, const double *bk, void *const *q,
                     int nq, hipStream_t st)
{
    const Geo &G = g->geo;
    const int n = g->n, nz = g->nz;
    constexpr int NF = RNF;
    const double ptop = g->p.ptop;
    RCoef C{};
    for (int K = 0; K <= nz; K++) {
        C.ak[K] = ak[K];
        C.bk[K] = bk[K];
    }
    fv3_status hs = run_halo_cells(g, &s->delp, 1, nz, 0, st);   // face winds read the neighbour cells
    if (hs != FV3_OK) return hs;
    const dim3 blk(256);
    // bytes of LDS of a block: interface pressures, coefficients; staged fields of a group
    auto lds = [&](const RBatch &B, int NF, int lw) {
        size_t most = 0;
        for (int f0 = 0; f0 < B.nf; f0 += NF) {
            size_t e = 0;
            for (int f = f0; f < std::min(f0 + NF, B.nf); f++)
                e += (size_t)(sizeof(T) == 8 || B.fp64[f] ? nz : (nz + 1) / 2) * 8 << lw;
            most = std::max(most, e);
        }
        return (((size_t)(nz + 1) * 8) << lw) + (size_t)(nz + 1) * 16 + most;
    };
    auto grid = [&](long cols, int planes, int lw) { return dim3((unsigned)((cols + (1 << lw) - 1) >> lw), (unsigned)planes); };
    const int lw = remap_shift(nz, (long)n * n * g->T);
    // winds at faces
    {
        RBatch B{};
        B.fld[0] = s->u;
        B.fld[1] = s->v;
        B.nf = 2;
        timed("k_remap_winds", k_remap<T, RM_WIND, 1>, lds(B, 1, lw), grid((long)n * (n + 1), g->T * 2, lw), blk, st, G, lw, ptop, C, B,
              (const T *)s->delp, g->flags);
    }
    // cell fields: pt, w, delz (as delz/delp), tracers.  A field listed again
    // is remapped once.  delp, if it is listed as a tracer, comes last and
    // alone: the blocks of every group of fields read it.
    std::vector<void *> fs = {s->pt, s->w, s->delz};
    bool own = false;
    for (int m = 0; m < nq; m++) {
        if (q[m] == s->delp) own = true;
        else if (std::find(fs.begin(), fs.end(), q[m]) == fs.end()) fs.push_back(q[m]);
    }
    auto cells = [&](void *const *f, int nf) {
        RBatch B{};
        B.nf = nf;
        for (int k = 0; k < nf; k++) {
            B.fld[k] = f[k];
            B.fp64[k] = B.ratio[k] = f[k] == (const void *)s->delz;
        }
        const int groups = (nf + NF - 1) / NF;
        timed("k_remap_cells", k_remap<T, RM_CELL, NF>, lds(B, NF, lw), grid((long)n * n, g->T * groups, lw), blk, st, G, lw, ptop, C, B,
              (const T *)s->delp, g->flags);
    };
    for (size_t b = 0; b < fs.size(); b += RFIELDS) cells(&fs[b], (int)std::min<size_t>(RFIELDS, fs.size() - b));
    if (own) cells(&s->delp, 1);
    timed("k_remap_delp", k_remap_delp<T>, ((size_t)(nz + 1) * 8) << lw, grid((long)n * n, g->T, lw), blk, st, G, lw, ptop, C, (T *)s->delp);
    return hipGetLastError() == hipSuccess ? FV3_OK : FV3_EDEVICE;
}

}  // namespace

fv3_status run_remap(fv3_state *s, const fv3_grid *g, const double *ak, const double *bk, void *const *q, int nq,
                     hipStream_t st)
{
    return g->bulk_bytes == 8 ? remap<double>(s, g, ak, bk, q, nq, st) : remap<float>(s, g, ak, bk, q, nq, st);
}

}  // namespace fv3
