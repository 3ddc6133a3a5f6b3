// c_sw (csw.hip, csw_edge.hip).
#pragma once

#include "march.hpp"

namespace fv3 {

// D-grid winds and cell fields in; C-grid winds, half-step cells and area
// fluxes out, all with filled halos in.
template <class B>
struct CswArgs {
    int strips, width, segs, rows;   // set by csw
    B dt2;
    const B *u, *v, *delp, *pt, *w;
    B *uc, *vc, *delpc, *ptc, *wc, *ax, *ay;
};
template <class B>
void csw(const fv3_grid *g, const CswArgs<B> &a, hipStream_t st);

// FP32 with one-sided stencils at tile edges (csw_edge.hip)
void csw_edge(const fv3_grid *g, const CswArgs<float> &a, hipStream_t st);

}  // namespace fv3
