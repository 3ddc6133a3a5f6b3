// Elimination of the column solves' tridiagonal system in chunks of layers
// (device code of column.hip; plain arithmetic, so that it can be checked on
// the host).
//
// Layer k with mass m couples to the layers above and below by A0 and A1
// (A0 = 0 at the top): diagonal m + A0 + A1, off-diagonals -A0, -A1.  The
// elimination carries e = 1 - c, c the ratio w_k = d_k + c_k w_{k+1}:
//
//   pivot = m + A0 e + A1,   c' = A1 / pivot,   e' = (m + A0 e) / pivot,
//
// sums and products of positive numbers only.  With c itself the pivot is
// m + A0 + A1 - A0 c, where for stiff columns (A much larger than m, c next
// to 1) the mass is what is left of a difference of large, nearly equal
// numbers.  Root mean square error of w against 128 bits (sigma layers,
// relative to the column's largest |w|), at 79 layers and a solve of 15 s /
// 512 layers and 15 s: 5.1e-17 / 3.4e-17; with c in the chunk's map 9.8e-16 /
// 8.7e-15, by a Thomas walk down all layers 3.8e-16 / 1.1e-15.
#pragma once
#include "flog.hpp"

namespace fv3 {

// A chunk's map of the e above it to the e below it, the quotient x / y of a
// linear map of (x, y) with non-negative entries, formed without a division
struct ElimMap {
    double m00 = 1.0, m10 = 0.0, m01 = 0.0, m11 = 1.0;
    __host__ __device__ inline void layer(double A0, double A1, double m)
    {
        m00 = A0 * m00 + m * m10;
        m01 = A0 * m01 + m * m11;
        m10 = m00 + A1 * m10;
        m11 = m01 + A1 * m11;
    }
    __host__ __device__ inline double operator()(double e) const { return fdiv(m00 * e + m01, m10 * e + m11); }
};

// One layer of the elimination.  e, d, q: of the layer above in, of this layer
// out (its own right-hand sides give d, the d above the chunk q times itself);
// returns c.
__host__ __device__ inline double elim_layer(double A0, double A1, double m, double rhs, double &e, double &d, double &q)
{
    const double s = m + A0 * e, rp = fdiv(1.0, s + A1);
    d = (rhs + A0 * d) * rp;
    q = A0 * rp * q;
    e = s * rp;
    return A1 * rp;
}

}  // namespace fv3
