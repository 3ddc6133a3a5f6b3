// Marching transport kernels (transport.hip).
#pragma once

#include "fv3_internal.hpp"

namespace fv3 {

constexpr int MARCH_TRACERS = 4;   // tracers per launch, at most (FP64: 3, for the registers)

// Arguments of one marching transport launch.
template <class T>
struct MarchArgs {
    int strips, width, segs, rows;         // strips of `width` columns, segments of `rows` rows per plane
    const T *q[MARCH_TRACERS];             // fields (MASS: delp, pt, w; WIND: absolute vorticity; TRACER)
    T *out[MARCH_TRACERS];
    const T *crx, *cry, *xfx, *yfx, *area;
    // MASS: accumulators
    double *mfx, *mfy;
    T *cxa, *cya;
    // MASS, TRACER: tile-edge fluxes of the fields (edge-flux fix-up, or null)
    T *FX[MARCH_TRACERS], *FY[MARCH_TRACERS];
    // WIND: kinetic energy, winds, 1/lengths, Coriolis term and coefficient of the vorticity damping
    const T *ke, *rdx, *rdy, *rdxc, *rdyc, *fc;
    T *u, *v;
    T nuv;
    // HEIGHT: interface heights; FP32: the reference heights are written to zref
    const double *z;
    double *zref;
    // TRACER: accumulated mass fluxes, of which a sub-cycle takes 1 / rs; layer
    // mass before the sub-cycle and (or null) after it; area
    const double *mx, *my, *dp1, *area64;
    double *dp2;
    double rs, rrs;
};

// fv_tp_2d of delp, pt and w with the mass fluxes of the first as weights of
// the others; fluxes and Courant numbers are added to the accumulators.
template <class T>
void march_mass(const fv3_grid *g, MarchArgs<T> a, hipStream_t st);
// vorticity fluxes and the D-grid wind update
template <class T>
void march_wind(const fv3_grid *g, MarchArgs<T> a, hipStream_t st);
// interface heights (advective form, interface-averaged Courant numbers)
template <class T>
void march_height(const fv3_grid *g, MarchArgs<T> a, hipStream_t st);
// nq tracers (at most MARCH_TRACERS, 3 in FP64) in one launch
template <class T>
void march_tracer(const fv3_grid *g, int nq, MarchArgs<T> a, hipStream_t st);

}  // namespace fv3
