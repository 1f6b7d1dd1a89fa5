// The weight of a solid in the blur zone (Lin, Derr & Rycroft, arXiv 2104.00095, main
// text eq. (sm_heavi) and eq. (mod_heaviside)): 1 - H_eps(phi0(x)), with the smoothed
// Heaviside of half-width eps.  Device code; the host test of the certificates compiles it
// over the HIP emulation.
#pragma once
#include "rmx_device.h"

namespace rmx {
namespace dev {

constexpr double kPi = 3.141592653589793;

__device__ __forceinline__ double heaviside_eps(double phi, double eps) {
    if (phi <= -eps) return 0.0;
    if (phi >= eps) return 1.0;
    return 0.5 * ((1.0 + phi / eps) + sin(kPi * phi / eps) / kPi);
}

// Whether H_eps(phi0(x)) is certainly 0 or 1: the weight 1 - H_eps of an ellipsoid then
// follows without the exact distance.  Where the distance from x to the surface is certainly
// at least eps, H_eps is exactly 0 or 1 whatever the exact phi0.  Three certificates, in body
// coordinates y with semi-axes a and r = eps (1 + 1e-9):
//  - with F = sum_i (y_i / a_i)^2 and g = |(y_i / a_i^2)|, the quadratic form over the ball
//    |v| <= r stays below F + 2 r g + r^2 / a_min^2 and above F - 2 r g (Cauchy-Schwarz on
//    its linear term), so the ball lies inside if the first is < 1 and outside if the
//    second is > 1;
//  - the cube |v_i| <= r around y, which holds that ball, lies outside the ellipsoid if
//    sum_i (max(|y_i| - r, 0) / a_i)^2 > 1 (the quadratic form grows with every |y_i|);
//  - with rho = |y / a|, the distance is at least (rho - 1) a_min outside (rho E contains the
//    ellipsoid grown by a ball of that radius) and (1 - rho) a_min inside.
// Each sum is compared with 1 -+ 1e-12 and each bound with r: margins far above the
// rounding of these few operations and of any exact distance.
__device__ __forceinline__ bool weight_certain(const ShapeR& s, double x0, double x1, double x2,
                                               double eps, double* w) {
#pragma clang fp contract(off)
    if (s.kind == 2 && finite3(x0, x1, x2)) {
        double y0, y1, y2;
        body(s, x0, x1, x2, y0, y1, y2);
        const double r = eps * (1.0 + 1e-9);
        const double amin = fmin(s.e0, fmin(s.e1, s.e2));
        const double q0 = y0 / s.e0, q1 = y1 / s.e1, q2 = y2 / s.e2;
        const double F = (q0 * q0 + q1 * q1) + q2 * q2;
        const double g0 = q0 / s.e0, g1 = q1 / s.e1, g2 = q2 / s.e2;
        const double gr = 2.0 * r * sqrt((g0 * g0 + g1 * g1) + g2 * g2);
        *w = 1.0;   // phi0 <= -eps
        if ((F + gr) + (r / amin) * (r / amin) < 1.0 - 1e-12) return true;
        *w = 0.0;   // phi0 >= eps
        if (F - gr > 1.0 + 1e-12) return true;
        const double u0 = fabs(y0), u1 = fabs(y1), u2 = fabs(y2);
        const double o0 = fmax(u0 - r, 0.0) / s.e0, o1 = fmax(u1 - r, 0.0) / s.e1,
                     o2 = fmax(u2 - r, 0.0) / s.e2;
        if ((o0 * o0 + o1 * o1) + o2 * o2 > 1.0 + 1e-12) return true;
        const double rho = sqrt(F);
        const double need = r + 1e-9 * amin * (rho + 1.0);
        if ((rho - 1.0) * amin >= need) return true;
        *w = 1.0;
        if ((1.0 - rho) * amin >= need) return true;
    }
    return false;
}

// 1 - H_eps(phi0(x)), the weight of a solid at x, from the exact distance where the
// certificates do not decide it.
__device__ __forceinline__ double weight_at(const ShapeR& s, double x0, double x1, double x2,
                                           double eps) {
    double w;
    if (weight_certain(s, x0, x1, x2, eps, &w)) return w;
    return 1.0 - heaviside_eps(phi0(s, x0, x1, x2), eps);
}

// The distance from body point y to the ellipsoid with semi-axes e by Newton's method on the
// closest point's multiplier s, the root of F(s) = sum_i (c_i / (s + d_i))^2 = 1, to
// rounding.  F^(-1/2) is increasing and concave in s, so its steps from the lower bound of
// the root approach the root from below, quadratically; they run in approximate arithmetic
// until a step is below 2^-30 of s, then two steps on F follow in full precision.  A
// coordinate of 0 is taken as a tiny one, which moves the distance by less than its
// rounding and keeps the root simple where the closest point leaves the coordinate plane.
// A point that is not finite has no distance: the shortest semi-axis, outside, as phi0 has
// for NaN.
// (The bisection that fixes phi0 bit for bit takes about ten times the operations, in a
// loop whose length depends on the point.)
__device__ __forceinline__ double distance_newton(double e0, double e1, double e2, double y0,
                                                  double y1, double y2) {
    if (!finite3(y0, y1, y2)) return fmin(e0, fmin(e1, e2));
    const double u0 = fmax(fabs(y0), 0x1p-180), u1 = fmax(fabs(y1), 0x1p-180),
                 u2 = fmax(fabs(y2), 0x1p-180);
    const double q0 = e0 * e0, q1 = e1 * e1, q2 = e2 * e2;
    const double qm = fmin(q0, fmin(q1, q2));
    const double d0 = q0 - qm, d1 = q1 - qm, d2 = q2 - qm;
    const double c0 = e0 * u0, c1 = e1 * u1, c2 = e2 * u2;
    // the root lies between a shortest axis' term alone and all terms over the shortest
    const double s0 = d0 == 0.0 ? c0 : (d1 == 0.0 ? c1 : c2);
    const double s1 = sqrt(fma(c0, c0, fma(c1, c1, c2 * c2)));
    double s = s0;
#pragma unroll 1
    for (int k = 0; k < 100; ++k) {
        const double i0 = rcp_refined(s + d0), i1 = rcp_refined(s + d1), i2 = rcp_refined(s + d2);
        const double t0 = c0 * i0, t1 = c1 * i1, t2 = c2 * i2;
        const double F = fma(t0, t0, fma(t1, t1, t2 * t2));
        const double G = fma(t0 * t0, i0, fma(t1 * t1, i1, (t2 * t2) * i2));
        double r = __builtin_amdgcn_rsq(F);
        r = r * (1.5 - (0.5 * F) * (r * r));   // F^(-1/2)
        const double step = (r - 1.0) * rcp_refined(G * (r * r * r));
        s = fmin(fmax(s - step, s0), s1);
        if (!(fabs(step) > 0x1p-30 * s)) break;
    }
    // The closest point is y_i q_i / (s + d_i), at y_i t / (s + d_i) from y with t = s - qm:
    // t carries the distance without cancellation near the surface.
    double t = s - qm;
    double i0 = 0.0, i1 = 0.0, i2 = 0.0;
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        i0 = rcp_newton2(s + d0);
        i1 = rcp_newton2(s + d1);
        i2 = rcp_newton2(s + d2);
        if (k == 2) break;
        const double t0 = c0 * i0, t1 = c1 * i1, t2 = c2 * i2;
        const double F = fma(t0, t0, fma(t1, t1, fma(t2, t2, -1.0)));
        const double G = fma(t0 * t0, i0, fma(t1 * t1, i1, (t2 * t2) * i2));
        const double step = 0.5 * F * rcp_refined(G);
        s = s + step;
        t = t + step;
    }
    const double v0 = u0 * i0, v1 = u1 * i1, v2 = u2 * i2;
    return fabs(t) * sqrt(fma(v0, v0, fma(v1, v1, v2 * v2)));
}

}  // namespace dev
}  // namespace rmx
