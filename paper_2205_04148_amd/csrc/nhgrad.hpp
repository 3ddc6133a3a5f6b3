// nh_p_grad (nhgrad.hip).
#pragma once

#include "march.hpp"

namespace fv3 {

// Pressure, geopotential (interfaces) and delp, all with filled halos; the
// D-grid winds take the pressure gradient over bdt.
template <class B>
struct NhArgs {
    int layers, strips, width, segs, rows;   // set by nh_grad
    double bdt;
    const double *pfull, *phi;
    const B *delp;
    B *u, *v;
};
template <class B>
void nh_grad(const fv3_grid *g, const NhArgs<B> &a, hipStream_t st);

}  // namespace fv3
