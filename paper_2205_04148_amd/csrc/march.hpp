// Common parts of the marching kernels: lane shifts, addressing and the split
// of a plane into strips and segments (gfx950).
#pragma once

#include "launch.hpp"

namespace fv3 {

// value of the lane to the west (l - 1) or east (l + 1); lanes without one get 0
template <int CTRL>
DEVI float lane_shift(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
DEVI double lane_shift(double x)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    const i2 v = __builtin_bit_cast(i2, x);
    i2 r;
    r.x = __builtin_amdgcn_update_dpp(0, v.x, CTRL, 0xf, 0xf, true);
    r.y = __builtin_amdgcn_update_dpp(0, v.y, CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, r);
}
template <class T>
DEVI T west(T x) { return lane_shift<0x138>(x); }   // wave shift right by one
template <class T>
DEVI T east(T x) { return lane_shift<0x130>(x); }   // wave shift left by one

DEVI float ffma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
DEVI double ffma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// element of a plane (block-uniform pointer to its halo corner) at byte offset o
template <class T>
DEVI T &el(T *plane, unsigned o) { return *(T *)((char *)plane + o); }

// Strips of at most 58 of `pts` columns, equally wide; segments of rows.  A
// segment marches `extra` rows more than it owns, so few long segments do the
// least work and many short ones spread over more of the 1024 SIMDs: the
// number of segments with the least (wavefronts on the fullest SIMD) x (rows
// marched), where a round of fewer than two wavefronts on a SIMD takes as long
// as one of two (they wait on each other's latency instead of sharing it) and
// occ wavefronts make a round.  FP64 wind update at C192 x 79 (three wavefronts
// fit): 365 us in 3 segments, 444 in 2 (a round of three wavefronts and one of
// a single one).
inline void march_shape(int pts, long planes, int extra, int occ, int &strips, int &width, int &segs, int &rows)
{
    strips = (pts + 57) / 58;
    width = (pts + strips - 1) / strips;
    long best = -1;
    for (int s = 1; s <= pts; s++) {
        const int rw = (pts + s - 1) / s;
        const long waves = (planes * strips * s + 1023) / 1024, last = waves % occ;
        const long cost = (10 * (waves - last) + (last == 0 ? 0 : last > 2 ? 10 * last : 22)) * (rw + extra);
        if (best < 0 || cost < best) {
            best = cost;
            rows = rw;
        }
        if (waves > 4 * occ) break;
    }
    segs = (pts + rows - 1) / rows;
}

}  // namespace fv3
