// The floating-point decisions of the distance-to-segment predicate
// (segdist.h), in plain arithmetic: no header or intrinsic of the device, so
// that its test compiles the same lines for the host.
#pragma once

#include <math.h>

namespace spade {

struct Seg {
    double ax, ay, bx, by;
};

// Whether a finite point is within distance r of segment s: within (1), not
// within (0), or open (-1: the exact test decides).  r2 = fl(r * r).  Without
// the exact test's calls a kernel needs half the registers (k_buf_bits: 64 for
// 128) and keeps twice the wavefronts.
//
// The nearest point is a, b or the foot of the perpendicular, chosen as the
// exact test does: by the sign of (p - a).(b - a) at a and of (p - b).(b - a)
// at b.  A rounded dot product of terms that each carry three roundings is off
// by at most 4 eps |p - a| |b - a| (eps = 2^-53), so the point lies at most
// 4 eps |p - a| along the segment beside where the sign puts it, and the
// squared distances of the two regions differ by less than 16 eps^2 of
// themselves; likewise at b.  (Both signs from the dot product at a, the
// second by comparison with |b - a|^2, would be off by 4 eps |b - a| at b:
// far more than the distance from b to a near point of a long segment.)
// Should both ends be taken for the nearer one, the segment is shorter than
// 8 eps of the distance.  The cross product is enclosed by its rounding bound
// as in perp_sign, and the margins of 1e-12 cover the rest; contraction into
// FMA only leaves roundings out.  Any product that could leave the normal
// range leaves the test open.
__device__ __forceinline__ int seg_near_filter(double px, double py, const Seg &s, double r2)
{
    const double ex = s.bx - s.ax, ey = s.by - s.ay;
    const double fx = px - s.bx, fy = py - s.by;
    double dx = px - s.ax, dy = py - s.ay;
    const double l2 = ex * ex + ey * ey;
    const bool past_a = dx * ex + dy * ey > 0.0, before_b = fx * ex + fy * ey < 0.0;
    double lo, hi, rhs = r2;
    if (past_a && before_b) {
        const double c1 = ex * dy, c2 = ey * dx;
        const double c = fabs(c1 - c2), ec = 6.7e-16 * (fabs(c1) + fabs(c2));
        const double a = fmax(c - ec, 0.0), b = c + ec;
        lo = a * a;
        hi = b * b;
        rhs = r2 * l2;
    } else {
        if (past_a) {
            dx = fx;
            dy = fy;
        }
        lo = hi = dx * dx + dy * dy;
    }
    if (!(rhs > 1e-250 && hi < 1e250 && l2 < 1e250)) return -1;
    if (hi * (1.0 + 1e-12) < rhs * (1.0 - 1e-12)) return 1;
    if (lo * (1.0 - 1e-12) > rhs * (1.0 + 1e-12)) return 0;
    return -1;
}

}  // namespace spade
