// Device indexing helpers and the kernel launch machinery shared by the
// substep path's translation units (gfx950).
#pragma once

#include <type_traits>
#include <utility>

#include "fv3_internal.hpp"

namespace fv3 {

#define DEVI __device__ __forceinline__

// ------------------------------------------------------------ indexing
DEVI long pidx(const Geo &G, int L, int t, int k) { return G.off0 + ((long)t * L + k) * G.lev; }
// Element (i, j) of a plane whose interior origin is P (i, j >= -3): the
// address is the plane's halo corner (-3, -3) plus a non-negative 32-bit
// byte offset, so that a block-uniform P becomes a scalar base with one
// 32-bit vector offset instead of per-lane 64-bit address arithmetic.
template <class T>
DEVI T &at_(T *p, int i, int j, int pitch)
{
    char *b = (char *)(p - (3 * pitch + 3));
    return *(T *)(b + (unsigned)((j + 3) * pitch + (i + 3)) * (unsigned)sizeof(T));
}
#define AT(P, i, j) at_((P), (int)(i), (int)(j), (int)G.pitch)

// a / b in the FP32 bulk through the hardware reciprocal (about 1 ulp, far
// below the FP32 bulk's rounding), FP64 exact
template <class T>
DEVI T rdiv(T a, T b)
{
    if constexpr (std::is_same<T, float>::value) return a * __builtin_amdgcn_rcpf(b);
    else return a / b;
}

DEVI int stx_(int st) { return (st == SC || st == SY) ? 1 : 0; }
DEVI int sty_(int st) { return (st == SC || st == SX) ? 1 : 0; }
DEVI int floor2(int a) { return a >= 0 ? (a >> 1) : -((1 - a) >> 1); }

DEVI bool in_corner(const Geo &G, int st, int i, int j)
{
    int x2 = 2 * i + stx_(st), y2 = 2 * j + sty_(st), n2 = 2 * G.n;
    return G.cube && (x2 < 0 || x2 > n2) && (y2 < 0 || y2 > n2);
}

// Corner view: the edge-halo point a corner-block point (i, j) of stagger st
// reads in sweep mode `mode` (0 x, 1 y); cw reports the rotation sense.
DEVI void corner_src(const Geo &G, int st, int i, int j, int mode, int &qi, int &qj, bool &cw)
{
    int n2 = 2 * G.n;
    int x2 = 2 * i + stx_(st), y2 = 2 * j + sty_(st);
    int vx = x2 < 0 ? 0 : n2, vy = y2 < 0 ? 0 : n2;
    int c = (x2 < 0 ? 0 : 1) + (y2 < 0 ? 0 : 2);
    cw = mode == 0 ? (c == 0 || c == 3) : (c == 1 || c == 2);
    int dx = x2 - vx, dy = y2 - vy;
    int qx2 = cw ? vx + dy : vx - dy;
    int qy2 = cw ? vy - dx : vy + dx;
    qi = floor2(qx2);
    qj = floor2(qy2);
}

// scalar read through the corner view
template <class T>
DEVI T sv(const Geo &G, const T *P, int st, int i, int j, int mode)
{
    if (in_corner(G, st, i, j)) {
        int qi, qj;
        bool cw;
        corner_src(G, st, i, j, mode, qi, qj, cw);
        return AT(P, qi, qj);
    }
    return AT(P, i, j);
}
// x component of a pair (X at stagger stx, Y its partner) through the view;
// sgn = false for unsigned pairs (lengths)
template <class T>
DEVI T pvx(const Geo &G, const T *X, const T *Y, int stx, int i, int j, int mode, bool sgn)
{
    if (in_corner(G, stx, i, j)) {
        int qi, qj;
        bool cw;
        corner_src(G, stx, i, j, mode, qi, qj, cw);
        T v = AT(Y, qi, qj);
        return (cw && sgn) ? -v : v;
    }
    return AT(X, i, j);
}
template <class T>
DEVI T pvy(const Geo &G, const T *X, const T *Y, int sty, int i, int j, int mode, bool sgn)
{
    if (in_corner(G, sty, i, j)) {
        int qi, qj;
        bool cw;
        corner_src(G, sty, i, j, mode, qi, qj, cw);
        T v = AT(X, qi, qj);
        return (!cw && sgn) ? -v : v;
    }
    return AT(Y, i, j);
}

DEVI bool is_vertex(const Geo &G, int i, int j)
{
    return G.cube && (i == 0 || i == G.n) && (j == 0 || j == G.n);
}

#define KBEGIN(L)                                                    \
    int i = ib + (int)(bk.x * blockDim.x + threadIdx.x);       \
    int j = jlo + (int)(bk.y * blockDim.y + threadIdx.y);      \
    if (i < ilo || i > ihi || j > jhi) return;                       \
    int t = (int)bk.z / (L), k = (int)bk.z % (L);        \
    (void)t; (void)k;

// Plane kernels: point range [ilo, ihi] x [jlo, jhi]; thread columns start at
// ib <= ilo, a multiple of 32 elements from the interior origin, so that every
// wavefront's 64 columns begin on a 128-byte line (interior column 0 is
// line-aligned in the layout).
#define KARGS Bk bk, int ib, int ilo, int ihi, int jlo, int jhi

template <class R>
struct Mets {
    const R *m[M_ALL];
};
typedef Mets<double> MetD;

// plane pointer of a 2-D metric for tile t
#define MP(M, name) ((M).m[name] + G.off0 + (long)t * G.lev)

// ---------------------------------------------------------- kernel launch
// Every kernel of the substep path is a device function that takes its block
// index explicitly.  It is launched either alone (k_one: the block index is
// the hardware one), or for an ensemble of grids in one launch (k_multi: grid
// z runs over the planes of all members, each block looks its member up in a
// small table and reads that member's arguments from device memory; blocks
// outside the member's own x/y extent exit at once).  Both paths run the same
// device code, so an ensemble member computes exactly what it computes alone.
template <class... A>
struct Tup;
template <>
struct Tup<> {
};
template <class H, class... R>
struct Tup<H, R...> {
    H h;
    Tup<R...> r;
};
static inline Tup<> tup() { return {}; }
template <class H, class... R>
static Tup<H, R...> tup(H h, R... r)
{
    return Tup<H, R...>{h, tup(r...)};
}
template <size_t I, class H, class... R>
DEVI const auto &tget(const Tup<H, R...> &t)
{
    if constexpr (I == 0) return t.h;
    else return tget<I - 1>(t.r);
}
template <auto F, class... A, size_t... I>
DEVI void tcall(Bk bk, const Tup<A...> &t, std::index_sequence<I...>)
{
    F(bk, tget<I>(t)...);
}

// MI355X hands consecutive workgroups of a launch to its eight XCDs in turn,
// and each XCD has its own L2.  The block index a kernel body sees is
// therefore permuted so that every XCD works on one contiguous range of the
// grid (x fastest, then y, then z): neighbouring tiles, which share halo
// lines, and the planes of one tile, which share the 2-D metric terms, then
// meet in the same L2.  The permutation is a bijection of the grid.
constexpr unsigned NXCD = 8;
DEVI Bk xcd_block()
{
    const unsigned gx = gridDim.x, gy = gridDim.y, total = gx * gy * gridDim.z;
    const unsigned id = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
    const unsigned q = total / NXCD, rem = total % NXCD, xcd = id % NXCD, local = id / NXCD;
    const unsigned lid = xcd * q + (xcd < rem ? xcd : rem) + local;
    return Bk{lid % gx, (lid / gx) % gy, lid / (gx * gy)};
}

// Minimum wavefronts per SIMD a kernel body is compiled for (its register
// budget: at most 512 / waves VGPRs); 1 leaves the choice to the compiler.
template <auto F>
constexpr int kocc = 1;

template <auto F, class... A>
__global__ void __launch_bounds__(256, kocc<F>) k_one(A... a)
{
    F(xcd_block(), a...);
}

template <auto F, class... A>
__global__ void __launch_bounds__(256, kocc<F>) k_multi(const Tup<A...> *__restrict__ args, const MemberBlk *__restrict__ tab,
                                               int members)
{
    // one-dimensional grid over every member's own blocks back to back (no
    // block outside a member's extent): find the member, then its block
    const int L = (int)xcd_block().x;
    int lo = 0, hi = members - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (tab[mid].b0 <= L) lo = mid;
        else hi = mid - 1;
    }
    const MemberBlk mb = tab[lo];
    const int gxy = mb.gx * mb.gy, local = L - mb.b0;
    if (gxy <= 0) return;
    const int bz = local / gxy, rem = local - bz * gxy, by = rem / mb.gx, bx = rem - by * mb.gx;
    if (bz >= mb.gz) return;
    tcall<F>(Bk{(unsigned)bx, (unsigned)by, (unsigned)bz}, args[lo], std::index_sequence_for<A...>{});
}

// Recording of the launch sequence of one call per member (ensemble mode).
extern thread_local Recorder *g_rec;   // defined in kernels.hip

template <class Tp>
static void rec_site(const char *name, const void *km, bool tunable, dim3 blk, int ex, int ey, int ez, const Tp &t)
{
    Recorder &R = *g_rec;
    if (R.member == 0) {
        Site s;
        s.name = name;
        s.kmulti = km;
        s.argsz = sizeof(Tp);
        s.tunable = tunable;
        s.blk = blk;
        R.sites.push_back(std::move(s));
    }
    if (R.pos >= R.sites.size() || R.sites[R.pos].kmulti != km) {
        R.bad = true;
        return;
    }
    Site &s = R.sites[R.pos++];
    const char *b = (const char *)&t;
    s.blob.insert(s.blob.end(), b, b + sizeof(Tp));
    s.ex.push_back(ex);
    s.ey.push_back(ey);
    s.ez.push_back(ez);
}

// plane kernels: 64 x 4 threads, one point each, grid z = planes
// Block shape of a plane kernel: 256 threads, bx consecutive points along i
// (a multiple of 16, so that a wavefront's row segments are whole 64-byte
// lines for FP32 and 128-byte lines for FP64).
struct Shape {
    int x, y;
};
constexpr Shape SH_DEFAULT{64, 4};

template <auto F, class... A>
static void launch2d_sh(const char *name, Shape sh, int ilo, int ihi, int jlo, int jhi, int planes,
                        hipStream_t st, A... a)
{
    // columns start at an aligned point: ilo itself, or -min(bx, 32) for halo ranges
    const int ib = ilo >= 0 ? ilo : -(sh.x < 32 ? sh.x : 32);
    if (g_rec) {
        rec_site(name, (const void *)k_multi<F, int, int, int, int, int, A...>, true, dim3(sh.x, sh.y, 1),
                 ihi - ib + 1, jhi - jlo + 1, planes, tup(ib, ilo, ihi, jlo, jhi, a...));
        return;
    }
    dim3 blk((unsigned)sh.x, (unsigned)sh.y, 1);
    dim3 grd((unsigned)((ihi - ib + sh.x) / sh.x), (unsigned)((jhi - jlo + sh.y) / sh.y), (unsigned)planes);
    bool tm = timing_wanted(name);
    TimingRec r;
    if (tm) timing_begin(name, st, r);
    hipLaunchKernelGGL((k_one<F, int, int, int, int, int, A...>), grd, blk, 0, st, ib, ilo, ihi, jlo, jhi, a...);
    if (tm) timing_end(st, r);
}
template <auto F, class... A>
static void launch2d_fn(const char *name, int ilo, int ihi, int jlo, int jhi, int planes, hipStream_t st, A... a)
{
    launch2d_sh<F>(name, SH_DEFAULT, ilo, ihi, jlo, jhi, planes, st, a...);
}
#define launch2d(kern, ...) launch2d_fn<kern>(#kern, __VA_ARGS__)
// with a block shape chosen per kernel (measured on MI355X at C192 x 79)
#define launch2d_s(kern, shape, ...) launch2d_sh<kern>(#kern, shape, __VA_ARGS__)

// generic launch with explicit shape (timed under `name`)
template <auto F, class... A>
static void launch_fn(const char *name, dim3 grd, dim3 blk, hipStream_t st, A... a)
{
    if (g_rec) {
        rec_site(name, (const void *)k_multi<F, A...>, false, blk, (int)grd.x, (int)grd.y, (int)grd.z, tup(a...));
        return;
    }
    bool tm = timing_wanted(name);
    TimingRec r;
    if (tm) timing_begin(name, st, r);
    hipLaunchKernelGGL((k_one<F, A...>), grd, blk, 0, st, a...);
    if (tm) timing_end(st, r);
}

}  // namespace fv3
