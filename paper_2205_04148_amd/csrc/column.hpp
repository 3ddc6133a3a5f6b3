// Column solves and interface heights (column.hip).
#pragma once

#include "fv3_internal.hpp"

namespace fv3 {

// Arguments of one column solve.  Arrays are fields in the grid's layout.
template <class B>
struct ColArgs {
    double dt, beta, ptop;
    int lw;                         // log2 of the columns per block (set by column_solve)
    int cubic;                      // interface perturbation: 0 mass-linear, 1 cubic
    const B *dpi, *theta, *w, *qv;  // layer mass, potential temperature, w, humidity (or null)
    const double *phis;             // surface geopotential (or null: flat)
    const double *z;                // site 0: interface heights, halo filled
    const B *ax, *ay;               // site 0: half-step area fluxes
    const void *zt;                 // site 1: transported interface heights (FP32: deviations from zref)
    const double *zref;             // site 1, FP32: reference height per (tile, interface)
    double *pfull, *phi;            // interface pressure and geopotential (out)
    B *w_out, *delp_out, *pt_out;   // site 1
    double *delz_out, *z_out;       // site 1: thicknesses (negative), interface heights
};

template <class B, int SITE>
void column_solve(const fv3_grid *g, const ColArgs<B> &a, hipStream_t st);
// interface heights of the interior cells from the thicknesses
void column_heights(const fv3_grid *g, const double *delz, const double *phis, double *z, hipStream_t st);

}  // namespace fv3
