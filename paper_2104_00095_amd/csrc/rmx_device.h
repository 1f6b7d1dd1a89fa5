// Device helpers of the launch chain (classification, labels, per-layer brick fits).
// Method: Lin, Derr & Rycroft (arXiv 2104.00095), section "Extrapolation of xi(x,t)" and
// SI "Weighting scheme for weighted least squares-based extrapolation", eq. (weight).
#pragma once
#include "rmx_internal.h"

namespace rmx {
namespace dev {

__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A load through the global address space.  Pointers read from the descriptors are
// generic, and generic (flat) loads may complete out of order with LDS accesses, so the
// compiler waits for all of them at once; global loads complete in issue order, and a
// use waits only for the loads issued before it.  (The host emulation of the kernels
// defines RMX_GLOBAL_AS away.)
#ifndef RMX_GLOBAL_AS
#define RMX_GLOBAL_AS __attribute__((address_space(1)))
#define RMX_CONST_AS __attribute__((address_space(4)))
// Product of two integers below 2^23 in magnitude (full rate; a 32-bit product is not).
__device__ __forceinline__ int mul24(int a, int b) { return __mul24(a, b); }
// 1/x and x^(-1/2) in single precision, as the hardware approximates them.
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsq_fast(float x) { return __builtin_amdgcn_rsqf(x); }
#else
inline float rcp_fast(float x) { return 1.0f / x; }
inline float rsq_fast(float x) { return 1.0f / sqrtf(x); }
#define RMX_CONST_AS
inline int mul24(int a, int b) { return a * b; }
#endif
template <typename T>
__device__ __forceinline__ T load_global(const T* p) {
    return *(const RMX_GLOBAL_AS T*)p;
}

// Data that no thread of the launch writes (descriptors, lists of an earlier kernel), read
// at addresses that are the same in every lane: through the constant address space the loads
// are scalar ones, and a value read once stays good across the kernel's stores.  (Generic
// loads of the descriptors are vector loads, repeated after every store.)
typedef const RMX_CONST_AS DevSolid DevSolidC;
__device__ __forceinline__ DevSolidC* const_solid(const DevSolid* solids, int s) {
    return (DevSolidC*)(solids + s);
}
template <typename T>
__device__ __forceinline__ T load_const(const T* p) {
    return *(const RMX_CONST_AS T*)p;
}
// A double known to be the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform_double(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)uniform_int((int)b), hi = (unsigned)uniform_int((int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The same for a word and a pointer.
__device__ __forceinline__ unsigned long long uniform_word(unsigned long long v) {
    const unsigned lo = (unsigned)uniform_int((int)v), hi = (unsigned)uniform_int((int)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    return reinterpret_cast<T*>(uniform_word(reinterpret_cast<unsigned long long>(p)));
}

// ------------------------------------------------------------------------------------
// phi0 and the interior predicate.  Evaluated without contraction, in the fixed order the
// interface documents, so that the interior decision and the normal's sign test are
// bit-identical to any other implementation of the same expressions.
// ------------------------------------------------------------------------------------
struct ShapeR {
    int kind;
    double c0, c1, c2;
    double e0, e1, e2;
    double r00, r01, r02, r10, r11, r12, r20, r21, r22;  // rot[b][a]
};

template <typename Solid>
__device__ __forceinline__ ShapeR load_shape(const Solid* d) {
    ShapeR s;
    s.kind = d->kind;
    s.c0 = d->centre[0]; s.c1 = d->centre[1]; s.c2 = d->centre[2];
    s.e0 = d->semi[0]; s.e1 = d->semi[1]; s.e2 = d->semi[2];
    s.r00 = d->rot[0]; s.r01 = d->rot[1]; s.r02 = d->rot[2];
    s.r10 = d->rot[3]; s.r11 = d->rot[4]; s.r12 = d->rot[5];
    s.r20 = d->rot[6]; s.r21 = d->rot[7]; s.r22 = d->rot[8];
    return s;
}

__device__ __forceinline__ double norm3(double a, double b, double c) {
#pragma clang fp contract(off)
    return sqrt((a * a + b * b) + c * c);
}

__device__ __forceinline__ bool finite3(double a, double b, double c) {
    return __builtin_isfinite(a) && __builtin_isfinite(b) && __builtin_isfinite(c);
}

__device__ __forceinline__ void body(const ShapeR& s, double v0, double v1, double v2,
                                     double& y0, double& y1, double& y2) {
#pragma clang fp contract(off)
    const double d0 = v0 - s.c0, d1 = v1 - s.c1, d2 = v2 - s.c2;
    y0 = (s.r00 * d0 + s.r10 * d1) + s.r20 * d2;
    y1 = (s.r01 * d0 + s.r11 * d1) + s.r21 * d2;
    y2 = (s.r02 * d0 + s.r12 * d1) + s.r22 * d2;
}

// phi0(xi) < 0: |xi - c|^2 < R^2 (sphere) or the quadratic form < 1 (ellipsoid).
__device__ __forceinline__ bool interior(const ShapeR& s, double v0, double v1, double v2) {
#pragma clang fp contract(off)
    if (!finite3(v0, v1, v2)) return false;
    if (s.kind == 1) {
        const double dx = v0 - s.c0, dy = v1 - s.c1, dz = v2 - s.c2;
        return ((dx * dx + dy * dy) + dz * dz) < s.e0 * s.e0;
    }
    double y0, y1, y2;
    body(s, v0, v1, v2, y0, y1, y2);
    const double q0 = y0 / s.e0, q1 = y1 / s.e1, q2 = y2 / s.e2;
    return ((q0 * q0 + q1 * q1) + q2 * q2) < 1.0;
}

__device__ __forceinline__ double pick3(int i, double a, double b, double c) {
    return i == 0 ? a : (i == 1 ? b : c);
}

// |x| within [2^-200, 2^200] (false for 0, NaN and infinities).
__device__ __forceinline__ bool mid_range(double x) {
    const double a = fabs(x);
    return a >= 0x1p-200 && a <= 0x1p200;
}

// a / b, correctly rounded, for a and b of mid_range magnitude: the reciprocal refined by
// two Newton steps, then one residual correction.  These are the steps of the hardware's
// division sequence, whose scale and fix-up steps change nothing for such operands (no
// exponent near an overflow or underflow bound, quotient within 2^+-400).  Written out,
// the divisions of one bisection step no longer wait on each other for the single
// condition register that the sequence's scale and fused-multiply-add steps share.
__device__ __forceinline__ double div_mid(double a, double b) {
    const double y0 = __builtin_amdgcn_rcp(b);
    const double y1 = fma(y0, fma(-b, y0, 1.0), y0);
    const double y2 = fma(y1, fma(-b, y1, 1.0), y1);
    const double q = a * y2;
    return fma(fma(-b, q, a), y2, q);
}

// f(s) = sum over the non-zero coordinates of (c_i / (s + d_i))^2, minus 1, in the
// bisection's arithmetic.
template <bool kMid>
__device__ __forceinline__ double ell_f(double sm, double c0, double c1, double c2, double d0,
                                        double d1, double d2, bool w0, bool w1, bool w2) {
#pragma clang fp contract(off)
    double f = 0.0;
    if (kMid) {
        // all three quotients at once (a term of a zero coordinate is formed and dropped);
        // f >= +0 throughout, so adding +0 for it changes nothing
        const double t0 = div_mid(c0, sm + d0), t1 = div_mid(c1, sm + d1),
                     t2 = div_mid(c2, sm + d2);
        f = f + (w0 ? t0 * t0 : 0.0);
        f = f + (w1 ? t1 * t1 : 0.0);
        f = f + (w2 ? t2 * t2 : 0.0);
    } else {
        if (w0) { const double t = c0 / (sm + d0); f = f + t * t; }
        if (w1) { const double t = c1 / (sm + d1); f = f + t * t; }
        if (w2) { const double t = c2 / (sm + d2); f = f + t * t; }
    }
    return f - 1.0;
}

// 1/x to a few ulps: the hardware reciprocal and one Newton step.
__device__ __forceinline__ double rcp_refined(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}

// Bisection of the multiplier on [s0, s1] until the midpoint equals an end of the bracket
// (or f is exactly 0, or not a number); w_i: coordinate i is non-zero.
//
// The computed f is non-increasing in s on [s0, s1]: each operation is correctly rounded
// and monotone in its operands there (s + d_i, d_i >= 0, grows with s; c_i / x with
// c_i >= 0 shrinks as x > 0 grows; t * t for t >= 0 and the sums grow with their
// operands).  So once f(a) > 0 has been computed, every midpoint sm <= a has f(sm) > 0
// and moves s0 without an evaluation; likewise sm >= b once f(b) < 0.  The midpoints, and
// so the final bracket, are those of evaluating every step.  a and b lie 2^-44 (relative)
// either side of a few Newton steps on g(s) = F(s)^(-1/2) - 1 (F = f + 1, close to
// linear in s), taken in approximate arithmetic, or 2^-24 out where the first probe
// missed; each is used only once its own f has the needed sign.
struct Bracket {
    double s0, s1;
};
template <bool kMid>
__device__ __forceinline__ Bracket ellipsoid_bisect(double c0, double c1, double c2, double d0,
                                                    double d1, double d2, bool w0, bool w1,
                                                    bool w2, double s0, double s1) {
#pragma clang fp contract(off)
    double s = s0;
    for (int k = 0; k < 6; ++k) {
        double F = 0.0, G = 0.0;   // F = sum t_i^2, G = sum t_i^2 / (s + d_i)
        if (w0) { const double y = rcp_refined(s + d0), t = c0 * y; F = F + t * t; G = G + (t * t) * y; }
        if (w1) { const double y = rcp_refined(s + d1), t = c1 * y; F = F + t * t; G = G + (t * t) * y; }
        if (w2) { const double y = rcp_refined(s + d2), t = c2 * y; F = F + t * t; G = G + (t * t) * y; }
        double r = __builtin_amdgcn_rsq(F);
        r = r * (1.5 - (0.5 * F) * (r * r));                   // F^(-1/2)
        const double step = (r - 1.0) * rcp_refined(G * (r * r * r));   // g / g'
        s = fmin(fmax(s - step, s0), s1);                      // (a NaN step leaves s0 or s1)
    }
    const double pa = fmax(s * (1.0 - 0x1p-44), s0), pb = fmin(s * (1.0 + 0x1p-44), s1);
    const double fa = ell_f<kMid>(pa, c0, c1, c2, d0, d1, d2, w0, w1, w2);
    const double fb = ell_f<kMid>(pb, c0, c1, c2, d0, d1, d2, w0, w1, w2);
    // Any point whose f is positive bounds the root from below, any with f negative from
    // above: a probe that landed on the other side of the root is a bound of the other
    // kind, and one probe 2^-24 out then looks for the missing one.  Without it such a
    // lane would evaluate every step on that side (and hold its wave there).
    double a = fa > 0.0 ? pa : -__builtin_huge_val();
    double b = fb < 0.0 ? pb : __builtin_huge_val();
    if (b == __builtin_huge_val()) {
        if (fb > 0.0) a = fmax(a, pb);
        const double pw = fmin(s * (1.0 + 0x1p-24), s1);
        if (ell_f<kMid>(pw, c0, c1, c2, d0, d1, d2, w0, w1, w2) < 0.0) b = pw;
    }
    if (a == -__builtin_huge_val()) {
        if (fa < 0.0) b = fmin(b, pa);
        const double pw = fmax(s * (1.0 - 0x1p-24), s0);
        if (ell_f<kMid>(pw, c0, c1, c2, d0, d1, d2, w0, w1, w2) > 0.0) a = pw;
    }
    for (int it = 0; it < 4096; ++it) {
        const double sm = 0.5 * (s0 + s1);
        if (sm <= s0 || sm >= s1) break;
        double f;
        if (sm <= a)
            f = 1.0;    // f(sm) >= f(a) > 0
        else if (sm >= b)
            f = -1.0;   // f(sm) <= f(b) < 0
        else
            f = ell_f<kMid>(sm, c0, c1, c2, d0, d1, d2, w0, w1, w2);
        if (f > 0.0) {
            s0 = sm;
        } else if (f < 0.0) {
            s1 = sm;
        } else {
            s0 = sm;
            s1 = sm;
            break;
        }
    }
    return {s0, s1};
}

// Distance from body point y to the ellipsoid with semi-axes e: Lagrange multiplier of
// the closest point measured from the pole of the shortest axis among the non-zero
// coordinates, bisected until the midpoint equals an end of the bracket; the off-plane
// candidate first when every shortest-axis coordinate is exactly zero.
__device__ inline double ellipsoid_distance(double e0, double e1, double e2, double y0, double y1,
                                     double y2) {
#pragma clang fp contract(off)
    const double u0 = fabs(y0), u1 = fabs(y1), u2 = fabs(y2);
    const double q0 = e0 * e0, q1 = e1 * e1, q2 = e2 * e2;
    int amin = 0;
    if (e1 < pick3(amin, e0, e1, e2)) amin = 1;
    if (e2 < pick3(amin, e0, e1, e2)) amin = 2;
    int m = -1;
    if (u0 > 0.0) m = 0;
    if (u1 > 0.0 && (m < 0 || e1 < pick3(m, e0, e1, e2))) m = 1;
    if (u2 > 0.0 && (m < 0 || e2 < pick3(m, e0, e1, e2))) m = 2;
    const double emin = pick3(amin, e0, e1, e2);
    if (m < 0) return emin;
    const double em = pick3(m, e0, e1, e2);
    const double qmin = pick3(amin, q0, q1, q2);
    if (em > emin) {
        double S = 0.0, D = 0.0;
        if (u0 > 0.0) {
            const double x = (q0 * u0) / (q0 - qmin);
            const double t = x / e0;
            S = S + t * t;
            D = D + (x - u0) * (x - u0);
        }
        if (u1 > 0.0) {
            const double x = (q1 * u1) / (q1 - qmin);
            const double t = x / e1;
            S = S + t * t;
            D = D + (x - u1) * (x - u1);
        }
        if (u2 > 0.0) {
            const double x = (q2 * u2) / (q2 - qmin);
            const double t = x / e2;
            S = S + t * t;
            D = D + (x - u2) * (x - u2);
        }
        if (S < 1.0) return sqrt(D + qmin * (1.0 - S));
    }
    const double qm = pick3(m, q0, q1, q2);
    const double d0 = q0 - qm, d1 = q1 - qm, d2 = q2 - qm;
    double sq = 0.0;
    if (u0 > 0.0) { const double p = e0 * u0; sq = sq + p * p; }
    if (u1 > 0.0) { const double p = e1 * u1; sq = sq + p * p; }
    if (u2 > 0.0) { const double p = e2 * u2; sq = sq + p * p; }
    double s0 = em * pick3(m, u0, u1, u2);
    double s1 = sqrt(sq);
    // Every midpoint lies in [s0, s1], so (rounding being monotone) every denominator
    // sm + d_i (d_i >= 0 where u_i > 0) lies between s0 + d_i and s1 + d_i.
    const double c0 = e0 * u0, c1 = e1 * u1, c2 = e2 * u2;
    const bool w0 = u0 > 0.0, w1 = u1 > 0.0, w2 = u2 > 0.0;
    const bool mid = (!w0 || (mid_range(c0) && mid_range(s0 + d0) && mid_range(s1 + d0))) &&
                     (!w1 || (mid_range(c1) && mid_range(s0 + d1) && mid_range(s1 + d1))) &&
                     (!w2 || (mid_range(c2) && mid_range(s0 + d2) && mid_range(s1 + d2)));
    const Bracket br = mid ? ellipsoid_bisect<true>(c0, c1, c2, d0, d1, d2, w0, w1, w2, s0, s1)
                           : ellipsoid_bisect<false>(c0, c1, c2, d0, d1, d2, w0, w1, w2, s0, s1);
    s0 = br.s0;
    s1 = br.s1;
    const double s = 0.5 * (s0 + s1);
    double D = 0.0;
    {
        const double x = (u0 > 0.0) ? (q0 * u0) / (s + d0) : 0.0;
        D = D + (x - u0) * (x - u0);
    }
    {
        const double x = (u1 > 0.0) ? (q1 * u1) / (s + d1) : 0.0;
        D = D + (x - u1) * (x - u1);
    }
    {
        const double x = (u2 > 0.0) ? (q2 * u2) / (s + d2) : 0.0;
        D = D + (x - u2) * (x - u2);
    }
    return sqrt(D);
}

// A positive double n units in the last place up.
__device__ __forceinline__ double ulps_up(double x, int n) {
    return __longlong_as_double(__double_as_longlong(x) + n);
}

// x within [2^-60, 2^60].
__device__ __forceinline__ bool near_one(double x) { return x >= 0x1p-60 && x <= 0x1p60; }

// a / b, correctly rounded as div_mid, from a reciprocal y of b to about 2^-30.
__device__ __forceinline__ double div_near(double a, double b, double y) {
    const double y2 = fma(y, fma(-b, y, 1.0), y);
    const double q = a * y2;
    return fma(fma(-b, q, a), y2, q);
}

// The distance of ellipsoid_distance, bit for bit, without following its bisection to the
// end.  The computed f does not increase (see ellipsoid_bisect), so the bisection ends where
// f goes from positive to negative: if that is between adjacent numbers, or at a single 0
// between them, it ends there whatever its path.  f at the seven numbers around a Newton
// estimate of the root (steps in single precision, then in double, then one on the computed f
// itself; reciprocals refined from one number to the next) settles it for most points.  A run
// of zeros is entered at the first midpoint that falls on it: those points follow the path, from
// the whole bracket, by comparisons with the run's ends alone.
// Returns false, with nothing computed, for coordinates of 0, magnitudes far from 1, and where
// 27 numbers on one side do not hold the change of sign.
// Bound by the latency of the chain (a wave's points take it together): 5.3 us for a wave's
// phi0 with nothing else on the card, maps read included, against 10 us for the bounds 2^-44
// either side of the root and the ten evaluations on the path below.
__device__ __forceinline__ bool ellipsoid_distance_near(double e0, double e1, double e2, double y0,
                                                        double y1, double y2, double* dist) {
#pragma clang fp contract(off)
    const double u0 = fabs(y0), u1 = fabs(y1), u2 = fabs(y2);
    // (with these every operand of the divisions below is of mid_range magnitude)
    if (!(near_one(u0) && near_one(u1) && near_one(u2) && near_one(e0) && near_one(e1) &&
          near_one(e2)))
        return false;
    const double q0 = e0 * e0, q1 = e1 * e1, q2 = e2 * e2;
    const bool m1 = e1 < e0, m2 = e2 < (m1 ? e1 : e0);
    const double qm = m2 ? q2 : (m1 ? q1 : q0);
    const double d0 = q0 - qm, d1 = q1 - qm, d2 = q2 - qm;
    const double c0 = e0 * u0, c1 = e1 * u1, c2 = e2 * u2;
    const double s0 = m2 ? c2 : (m1 ? c1 : c0);
    const double s1 = sqrt((c0 * c0 + c1 * c1) + c2 * c2);
    // Newton steps on g(s) = F(s)^(-1/2) - 1 (F = f + 1) from the root of a point on the
    // surface: g grows and is concave, so from the first step on the root is approached from
    // below.  In units of qm first.
    float pf = 1.0f;
    {
        const double iq = rcp_refined(qm);
        const float D0 = (float)(d0 * iq), D1 = (float)(d1 * iq), D2 = (float)(d2 * iq);
        const float C0 = (float)(c0 * iq), C1 = (float)(c1 * iq), C2 = (float)(c2 * iq);
        const float S0 = (float)(s0 * iq);
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            const float i0 = rcp_fast(pf + D0), i1 = rcp_fast(pf + D1), i2 = rcp_fast(pf + D2);
            const float t0 = C0 * i0, t1 = C1 * i1, t2 = C2 * i2;
            const float a0 = t0 * t0, a1 = t1 * t1, a2 = t2 * t2;
            const float F = (a0 + a1) + a2, G = fmaf(a0, i0, fmaf(a1, i1, a2 * i2));
            const float r = rsq_fast(F);
            pf = fmaxf(pf - (r - 1.0f) * rcp_fast(G * (r * r * r)), S0);
        }
    }
    double p = fmax(qm * (double)pf, s0), G = 0.0;
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
        const double i0 = rcp_refined(p + d0), i1 = rcp_refined(p + d1), i2 = rcp_refined(p + d2);
        const double t0 = c0 * i0, t1 = c1 * i1, t2 = c2 * i2;
        const double a0 = t0 * t0, a1 = t1 * t1, a2 = t2 * t2;
        const double F = (a0 + a1) + a2;
        G = fma(a0, i0, fma(a1, i1, a2 * i2));   // sum t_i^2 / (s + d_i)
        double r = __builtin_amdgcn_rsq(F);
        r = r * fma(-0.5 * F, r * r, 1.5);                              // F^(-1/2)
        const double step = (r - 1.0) * rcp_refined(G * (r * r * r));   // g / g'
        p = fmax(p - step, s0);
        if (!(fabs(step) > 0x1p-18 * p)) break;
    }
    // one step on the computed f itself
    const double i0 = rcp_refined(p + d0), i1 = rcp_refined(p + d1), i2 = rcp_refined(p + d2);
    auto eval = [&](double s) {
        const double t0 = div_near(c0, s + d0, i0), t1 = div_near(c1, s + d1, i1),
                     t2 = div_near(c2, s + d2, i2);
        return ((t0 * t0 + t1 * t1) + t2 * t2) - 1.0;
    };
    p = p + 0.5 * eval(p) * rcp_refined(G);
    if (!(p > 0.0 && ulps_up(p, -40) > s0 && ulps_up(p, 40) < s1)) return false;
    int pos = 0, neg = 0, lo = -3, hi = 3;   // signs of f at p + lo..hi units
#pragma unroll
    for (int k = -3; k <= 3; ++k) {
        const double f = eval(ulps_up(p, k));
        pos += f > 0.0;
        neg += f < 0.0;
    }
#pragma unroll 1
    for (int n = 0; n < 8 && (pos == 0 || neg == 0); ++n) {   // three more, where one is missing
        const int from = pos == 0 ? lo - 3 : hi + 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double f = eval(ulps_up(p, from + k));
            pos += f > 0.0;
            neg += f < 0.0;
        }
        if (from < lo) lo = from; else hi = from + 2;
    }
    if (pos == 0 || neg == 0) return false;
    const double a = ulps_up(p, lo - 1 + pos), b = ulps_up(p, hi + 1 - neg);   // the run's ends
    const int zeros = hi - lo + 1 - pos - neg;
    double sm = zeros == 0 ? 0.5 * (a + b) : ulps_up(a, 1);
    if (zeros > 1) {
        // 0.5 (s0 + s1) from halved ends, which are exact; a midpoint on the run stays
        double h0 = 0.5 * s0, h1 = 0.5 * s1;
        sm = h0 + h1;
        int n = 0;
#pragma unroll 1
        do {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double h = 0.5 * sm;
                h0 = sm <= a ? h : h0;
                h1 = sm >= b ? h : h1;
                sm = h0 + h1;
            }
        } while ((sm <= a || sm >= b) && ++n < 256);
        if (sm <= a || sm >= b) return false;
    }
    const double x0 = div_near(q0 * u0, sm + d0, i0), x1 = div_near(q1 * u1, sm + d1, i1),
                 x2 = div_near(q2 * u2, sm + d2, i2);
    double D = (x0 - u0) * (x0 - u0);
    D = D + (x1 - u1) * (x1 - u1);
    D = D + (x2 - u2) * (x2 - u2);
    *dist = sqrt(D);
    return true;
}

// phi0 of a sphere: the operations of phi0's sphere branch below, without the ellipsoid
// code (whose registers a sphere-only kernel then does not hold).
__device__ __forceinline__ double phi0_sphere(const ShapeR& s, double v0, double v1, double v2) {
#pragma clang fp contract(off)
    const double dx = v0 - s.c0, dy = v1 - s.c1, dz = v2 - s.c2;
    const double dist = fabs(sqrt((dx * dx + dy * dy) + dz * dz) - s.e0);
    const bool in = finite3(v0, v1, v2) && ((dx * dx + dy * dy) + dz * dz) < s.e0 * s.e0;
    return in ? -dist : dist;
}

// Signed distance phi0(v), negative inside; the sign is the interior predicate's.
__device__ inline double phi0(const ShapeR& s, double v0, double v1, double v2) {
#pragma clang fp contract(off)
    double dist;
    if (s.kind == 1) {
        const double dx = v0 - s.c0, dy = v1 - s.c1, dz = v2 - s.c2;
        dist = fabs(sqrt((dx * dx + dy * dy) + dz * dz) - s.e0);
    } else {
        double y0, y1, y2;
        body(s, v0, v1, v2, y0, y1, y2);
        if (!ellipsoid_distance_near(s.e0, s.e1, s.e2, y0, y1, y2, &dist))
            dist = ellipsoid_distance(s.e0, s.e1, s.e2, y0, y1, y2);
    }
    return interior(s, v0, v1, v2) ? -dist : dist;
}

// ------------------------------------------------------------------------------------
// Helpers.
// ------------------------------------------------------------------------------------
// The last i in [0, n) with key(i) <= v (key ascending, key(0) <= v; v the same in every lane),
// by a whole wave: 64 keys at a time, so that up to 64 solids take one load's latency (a
// binary search waits for one load after the other: 0.3 to 1.4 us more per kernel, e.g. the H
// fill of 40 solids 13.5 against 12.1 us).
template <typename Key>
__device__ __forceinline__ int wave_search(int n, int64_t v, Key key) {
    const int lane = threadIdx.x & 63;
    int base = 0, len = n;
    while (len > 1) {   // uniform
        const int step = (len + 63) / 64, at = lane * step;
        bool le = false;
        if (at < len) le = key(base + at) <= v;
        const int skip = (__popcll(__ballot(le)) - 1) * step;
        base += skip;
        len = min(step, len - skip);
    }
    return uniform_int(base);
}
__device__ __forceinline__ int find_solid_by_chunk(const DevSolid* s, int n, int c) {
    return wave_search(n, c, [s](int i) { return (int64_t)load_global(&s[i].chunk_base); });
}

// Exclusive scan of one int per thread over a block of NW waves.
template <int NW>
__device__ __forceinline__ void block_scan(int v, int& excl, int& total, int* s_wave) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[wid] = x;
    __syncthreads();
    int wb = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int t = s_wave[i];
        if (i < wid) wb += t;
        tot += t;
    }
    excl = wb + x - v;
    total = tot;
    __syncthreads();
}

// Entries [0, count) of a list, split into one contiguous range per XCD (workgroups are dealt to
// the XCDs round-robin): neighbouring entries, whose halos overlap, are then fetched into one L2,
// and no block takes more than ceil(count / blocks) entries.  The ranges are equal where that
// holds for them, and in proportion to the XCDs' blocks elsewhere: equal ranges would give some
// blocks of a grid that is no multiple of 8 an entry too many (a lone 24^3 box, 27 blocks, 75 us
// per call against 60), and the other form costs short kernels more than its divisions (stress
// of 27 overlapping boxes, 290 tiles on 343 blocks, 113 us against 104).  The calling block takes
// begin, begin + stride, ... below end.
struct XcdRange {
    int begin, end, stride;
};
__device__ __forceinline__ XcdRange xcd_range(int count) {
    const int G = gridDim.x, b = blockIdx.x;
    const int x = b % kXcds;
    if (G % kXcds == 0 || count <= G - G % kXcds) {   // as many blocks each, or one entry a block
        const int per = (count + kXcds - 1) / kXcds;
        return {x * per + b / kXcds, min(count, (x + 1) * per), G / kXcds};
    }
    // Whole rounds of the grid, then one entry more for as many blocks as are left over, dealt
    // over the XCDs as the blocks are.
    const int rounds = count < G ? 0 : count / G, rest = count - rounds * G;
    const int before = x * (G / kXcds) + min(x, G % kXcds);   // blocks of the XCDs before
    const int mine = G / kXcds + (x < G % kXcds ? 1 : 0);
    const int lo = rounds * before + x * (rest / kXcds) + min(x, rest % kXcds);
    const int hi = lo + rounds * mine + rest / kXcds + (x < rest % kXcds ? 1 : 0);
    return {lo + b / kXcds, hi, mine};
}

// The same value, through an identity lane move the compiler cannot see through: work
// derived from it stays where it is written instead of being hoisted out of a loop and
// kept live (spilled) across the loop body.  All lanes of each quad must be active.
__device__ __forceinline__ int opaque_lane_value(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0xE4, 0xf, 0xf, false);   // quad_perm [0,1,2,3]
}

// 12 labels along a row as bits: data (label in [0, l)) and cells of layer l.  base:
// the box index of the row's column 0, which may lie up to 12 before the box row's first
// cell; columns outside [0, n0) give no bit.  One 16-byte load at any alignment holds the row and
// two labels more on each side (so that the address is a multiple of 4 where n0 is); near
// the ends of the array the window is moved inside it and the bits shifted back.
constexpr int kRowBits = 12;
struct RowBits {
    unsigned data, target;
};
struct __attribute__((packed, aligned(1))) Labels16 {
    uint32_t w[4];
};

// Bits 7, 15, 23, 31 of x as a nibble (the products never overlap in bits 21..24).
__device__ __forceinline__ unsigned high_bits(unsigned x) {
    return (((x & 0x80808080u) >> 7) * 0x00204081u >> 21) & 15u;
}

__device__ __forceinline__ RowBits label_row_bits(const int8_t* __restrict__ labels, int nc,
                                                  int base, int ox, int n0, int l) {
    const int lo = max(0, -ox), hi = min(kRowBits, n0 - ox);
    const unsigned valid = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    unsigned below = 0u, upto = 0u;   // labels in [0, l) and in [0, l], bit i: column i
    if (nc >= 16) {
        const int a = base - 2, w = min(max(a, 0), nc - 16);
        const auto* v = (const RMX_GLOBAL_AS Labels16*)(labels + w);
        // (b | 0x80) - l has its high bit clear only where the low seven bits of b are below
        // l (no byte borrows from the next); a byte with its own high bit set is negative
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned b = v->w[u], q = b | 0x80808080u;
            below |= high_bits(~((q - 0x01010101u * (unsigned)l) | b)) << (4 * u);
            upto |= high_bits(~((q - 0x01010101u * (unsigned)(l + 1)) | b)) << (4 * u);
        }
        // column j lies at window place a - w + 2 + j, with -14 <= a - w <= 15
        const int sh = a - w + 18;
        below = (unsigned)(((unsigned long long)below << 16) >> sh);
        upto = (unsigned)(((unsigned long long)upto << 16) >> sh);
    } else {
        for (int j = lo; j < hi; ++j) {
            const int lab = load_global(labels + base + j);
            below |= (lab >= 0 && lab < l) ? 1u << j : 0u;
            upto |= (lab >= 0 && lab <= l) ? 1u << j : 0u;
        }
    }
    return {below & valid, upto & ~below & valid};
}

// ------------------------------------------------------------------------------------
// Extrapolation of one layer.  A group of 4, 8 or 16 aligned lanes per band cell.
// ------------------------------------------------------------------------------------

template <typename T>
struct Moments {
    T m[10];   // sum w [1,d][1,d]^T: (0,0) (0,x) (0,y) (0,z) (x,x) (x,y) (x,z) (y,y) (y,z) (z,z)
    T r[12];   // sum w [1,d] v^T: rows 1, dx, dy, dz; columns the 3 components
    int g[5];  // unweighted integer moments over the positive-weight offsets, two 16-bit
               // fields per word: (n, sxx) (sx, sxy) (sy, sxz) (sz, syy) (syz, szz)
};

template <typename T>
__device__ __forceinline__ void zero(Moments<T>& a) {
#pragma unroll
    for (int q = 0; q < 10; ++q) a.m[q] = T(0);
#pragma unroll
    for (int q = 0; q < 12; ++q) a.r[q] = T(0);
#pragma unroll
    for (int q = 0; q < 5; ++q) a.g[q] = 0;
}

// Sums over aligned groups of 4, 8 or 16 lanes by DPP moves within a row: swap
// neighbours, swap pairs, then mirror the half-row (8) and the row (16).  Every lane of a
// group ends with the same, commutatively formed, sum.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ int dpp_v(int v) {
    return dpp_i<CTRL>(v);
}
template <int CTRL>
__device__ __forceinline__ double dpp_v(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = dpp_i<CTRL>((int)b), hi = dpp_i<CTRL>((int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                            (unsigned)lo));
}
template <int CTRL>
__device__ __forceinline__ float dpp_v(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}

template <int CTRL, int N, typename T>
__device__ __forceinline__ void reduce_step(T* a) {
#pragma unroll
    for (int q = 0; q < N; ++q) a[q] += dpp_v<CTRL>(a[q]);
}

// (sh: log2 of the group's lanes, 2, 3 or 4, the same in the whole block)
template <int N, typename T>
__device__ __forceinline__ void reduce_values(T* a, int sh) {
    reduce_step<0xB1, N>(a);                 // quad_perm [1,0,3,2]
    reduce_step<0x4E, N>(a);                 // quad_perm [2,3,0,1]
    if (sh >= 3) reduce_step<0x141, N>(a);   // row_half_mirror
    if (sh >= 4) reduce_step<0x140, N>(a);   // row_mirror
}

template <typename T>
__device__ __forceinline__ void reduce_lanes(Moments<T>& a, int sh) {
    reduce_values<10>(a.m, sh);
    reduce_values<12>(a.r, sh);
    reduce_values<5>(a.g, sh);
}

// Two signed 16-bit sums packed as lo + hi * 2^16 (|sums| < 2^15 for r <= 4).
__device__ __forceinline__ void unpack2(int p, long long& lo, long long& hi) {
    const int l = (int)(short)(p & 0xffff);
    lo = l;
    hi = (long long)((p - l) >> 16);
}

// Exact determinant of the integer Gram matrix of [1, d] over the positive-weight offsets
// (Laplace expansion by the 2x2 minors of rows 0,1 and rows 2,3).  For r <= 4 the entries
// are below 729 * 16 in magnitude, so every product fits in int64.
__device__ __forceinline__ long long det_gram(const int* gp) {
    long long n, sxx, sx, sxy, sy, sxz, sz, syy, syz, szz;
    unpack2(gp[0], n, sxx);
    unpack2(gp[1], sx, sxy);
    unpack2(gp[2], sy, sxz);
    unpack2(gp[3], sz, syy);
    unpack2(gp[4], syz, szz);
    const long long a0 = n, a1 = sx, a2 = sy, a3 = sz;
    const long long b0 = sx, b1 = sxx, b2 = sxy, b3 = sxz;
    const long long c0 = sy, c1 = sxy, c2 = syy, c3 = syz;
    const long long d0 = sz, d1 = sxz, d2 = syz, d3 = szz;
    const long long s0 = a0 * b1 - a1 * b0, s1 = a0 * b2 - a2 * b0, s2 = a0 * b3 - a3 * b0;
    const long long s3 = a1 * b2 - a2 * b1, s4 = a1 * b3 - a3 * b1, s5 = a2 * b3 - a3 * b2;
    const long long t5 = c2 * d3 - c3 * d2, t4 = c1 * d3 - c3 * d1, t3 = c1 * d2 - c2 * d1;
    const long long t2 = c0 * d3 - c3 * d0, t1 = c0 * d2 - c2 * d0, t0 = c0 * d1 - c1 * d0;
    return s0 * t5 - s1 * t4 + s2 * t3 + s3 * t2 - s4 * t1 + s5 * t0;
}

// 1 / x to within an ulp for x of mid_range magnitude.
__device__ __forceinline__ double rcp_newton2(double x) {
    const double y0 = __builtin_amdgcn_rcp(x);
    const double y1 = fma(y0, fma(-x, y0, 1.0), y0);
    return fma(y1, fma(-x, y1, 1.0), y1);
}

// Intercept of the WLS fit of one component from the normal equations M [b0 bx by bz] = R
// (M as in Moments::m), in FP64.  certain: every pivot is above 1e-4 of its diagonal, so M
// is certainly not singular where its entries are exact to c u, u the rounding unit of FP64
// and c about 100: the error of a pivot grows at most by the inverse of the pivots before
// it, to 100 u 1e8 of the diagonal at the last.
struct Intercept {
    double value;
    bool certain;
};
constexpr double kPivotTol = 1e-4;

// FP64 moments: the slopes eliminated from the last on (four reciprocals, no square root).
__device__ __forceinline__ Intercept solve_eliminate(const double* M, double r0, double r1,
                                                     double r2, double r3) {
    const double i3 = rcp_newton2(M[9]);
    const double f0 = M[3] * i3, f1 = M[6] * i3, f2 = M[8] * i3;
    const double m0 = fma(-f0, M[3], M[0]), m1 = fma(-f0, M[6], M[1]), m2 = fma(-f0, M[8], M[2]);
    const double m4 = fma(-f1, M[6], M[4]), m5 = fma(-f1, M[8], M[5]), m7 = fma(-f2, M[8], M[7]);
    const double p0 = fma(-f0, r3, r0), p1 = fma(-f1, r3, r1), p2 = fma(-f2, r3, r2);
    const double i2 = rcp_newton2(m7);
    const double h0 = m2 * i2, h1 = m5 * i2;
    const double n0 = fma(-h0, m2, m0), n1 = fma(-h0, m5, m1), n4 = fma(-h1, m5, m4);
    const double q0 = fma(-h0, p2, p0), q1 = fma(-h1, p2, p1);
    const double k0 = n1 * rcp_newton2(n4);
    const double k = fma(-k0, n1, n0);
    return {fma(-k0, q1, q0) / k, M[9] > kPivotTol * M[0] && m7 > kPivotTol * M[7] &&
                                      n4 > kPivotTol * M[4] && k > kPivotTol * M[0]};
}

// FP32 moments: Cholesky.  (Their rounding can leave M close to singular, and the value then
// depends on the way it is solved.)
__device__ __forceinline__ Intercept solve_cholesky(const double* M, double r0, double r1,
                                                    double r2, double r3) {
    const double l00 = sqrt(M[0]);
    const double i00 = 1.0 / l00;
    const double l10 = M[1] * i00, l20 = M[2] * i00, l30 = M[3] * i00;
    const double p1 = M[4] - l10 * l10;
    const double l11 = sqrt(p1);
    const double i11 = 1.0 / l11;
    const double l21 = (M[5] - l20 * l10) * i11, l31 = (M[6] - l30 * l10) * i11;
    const double p2 = M[7] - l20 * l20 - l21 * l21;
    const double l22 = sqrt(p2);
    const double i22 = 1.0 / l22;
    const double l32 = (M[8] - l30 * l20 - l31 * l21) * i22;
    const double p3 = M[9] - l30 * l30 - l31 * l31 - l32 * l32;
    const double l33 = sqrt(p3);
    const double i33 = 1.0 / l33;
    const double y0 = r0 * i00;
    const double y1 = (r1 - l10 * y0) * i11;
    const double y2 = (r2 - l20 * y0 - l21 * y1) * i22;
    const double y3 = (r3 - l30 * y0 - l31 * y1 - l32 * y2) * i33;
    const double b3 = y3 * i33;
    const double b2 = (y2 - l32 * b3) * i22;
    const double b1 = (y1 - l21 * b2 - l31 * b3) * i11;
    return {(y0 - l10 * b1 - l20 * b2 - l30 * b3) * i00,
            M[0] > 0.0 && p1 > kPivotTol * M[4] && p2 > kPivotTol * M[7] && p3 > kPivotTol * M[9]};
}

template <typename T>
__device__ __forceinline__ Intercept solve_intercept(const double* M, double r0, double r1,
                                                     double r2, double r3) {
    return sizeof(T) == 4 ? solve_cholesky(M, r0, r1, r2, r3) : solve_eliminate(M, r0, r1, r2, r3);
}

// 1 / |d| for |d|^2 = 0..48 (offsets within radius 4).
static __constant__ double c_rlen[49] = {
    0.0, 1.0, 0.70710678118654752, 0.57735026918962576, 0.5, 0.44721359549995794,
    0.40824829046386302, 0.37796447300922723, 0.35355339059327376, 0.33333333333333333,
    0.31622776601683793, 0.30151134457776362, 0.28867513459481288, 0.27735009811261456,
    0.26726124191242438, 0.25819888974716113, 0.25, 0.24253562503633297,
    0.23570226039551584, 0.22941573387056177, 0.22360679774997897, 0.21821789023599238,
    0.21320071635561044, 0.20851441405707477, 0.20412414523193151, 0.2,
    0.19611613513818404, 0.19245008972987526, 0.18898223650461362, 0.18569533817705186,
    0.18257418583505538, 0.17960530202677491, 0.17677669529663688, 0.17407765595569785,
    0.17149858514250883, 0.16903085094570331, 0.16666666666666667, 0.16439898730535729,
    0.16222142113076254, 0.16012815380508713, 0.15811388300841897, 0.15617376188860607,
    0.15430334996209191, 0.15249857033260467, 0.15075567228888181, 0.14907119849998598,
    0.14744195615489714, 0.14586499149789456, 0.14433756729740644};

// 1 / |(fx rho_0, fy rho_1, fz rho_2)| (out of line: the rare path of unequal spacings
// keeps its registers to itself).
static __device__ __noinline__ double rlen_scaled(const double* rho, double fx, double fy, double fz) {
    return 1.0 / norm3(fx * rho[0], fy * rho[1], fz * rho[2]);
}

struct CellCtx {
    int i, j, k, n0, n1, n2, le;
    int64_t ncell;
    const double* __restrict__ xi;
    const int8_t* __restrict__ labels;
    double a0, a1, a2;            // xi of the anchor datum
    double g0, g1, g2, rgn;       // normal (unnormalised) and 1/|g / rho|
    const double* rho;            // the solid's spacing ratios; null when they are equal
};

// Accumulate, from global memory, the moments of the eligible data within Chebyshev
// radius r <= 4 (radii beyond the staged halo, and r_s other than it).  The (2r+1)^2 rows
// (dy, dz) of the box are dealt to the nl lanes of the cell.  Eq. (weight):
// w = 2^-(|dx|+|dy|+|dz|), times the cosine between x_e - x_d =
// -(dx rho_x, dy rho_y, dz rho_z) h and the normal when use_normal; data with
// (dx gx + dy gy) + dz gz >= 0 (that exact expression, no contraction) get weight 0.
// Bound by the latency of its loads and, for the few waves that come here, of its instructions:
// a row's labels are one 16-byte load turned into bits, only its data are visited, and the next
// one's xi is on its way while one is added (in one copy of the code).
template <typename T>
__device__ __forceinline__ void gather_any(const CellCtx& cx, int r, bool use_normal, int lq,
                                           int nl, Moments<T>& acc) {
    const int D = 2 * r + 1;
#pragma unroll 1
    for (int row = lq; row < D * D; row += nl) {
        const int dz = row / D - r, dy = row - (dz + r) * D - r;
        const int jj = cx.j + dy, kk = cx.k + dz;
        if ((unsigned)jj >= (unsigned)cx.n1 || (unsigned)kk >= (unsigned)cx.n2) continue;
        const int first = (kk * cx.n1 + jj) * cx.n0 + cx.i - r;   // the box index of dx = -r
        unsigned data = label_row_bits(cx.labels, (int)cx.ncell, first, cx.i - r, cx.n0,
                                       cx.le).data & ((1u << D) - 1u);
        if (data == 0u) continue;
        const int dyz2 = dy * dy + dz * dz, ayz = abs(dy) + abs(dz);
        int dx = __builtin_ctz(data) - r;
        const double* p = cx.xi + (first + r);
        double x0 = load_global(p + dx), x1 = load_global(p + cx.ncell + dx),
               x2 = load_global(p + 2 * cx.ncell + dx), rl = c_rlen[dx * dx + dyz2];
#pragma unroll 1
        for (;;) {
            data &= data - 1u;
            const int nx = data ? __builtin_ctz(data) - r : dx;
            const double n0 = load_global(p + nx), n1 = load_global(p + cx.ncell + nx),
                         n2 = load_global(p + 2 * cx.ncell + nx), nrl = c_rlen[nx * nx + dyz2];
            const double fx = (double)dx, fy = (double)dy, fz = (double)dz;
            double ww = ldexp(1.0, -(abs(dx) + ayz));
            bool on = true;
            if (use_normal) {
#pragma clang fp contract(off)
                const double dot = (fx * cx.g0 + fy * cx.g1) + fz * cx.g2;
                on = dot < 0.0;
                if (cx.rho) rl = 1.0 / norm3(fx * cx.rho[0], fy * cx.rho[1], fz * cx.rho[2]);
                ww = (-dot * rl * cx.rgn) * ww;
            }
            if (on) {
                const T tw = (T)ww, tx = (T)fx, ty = (T)fy, tz = (T)fz;
                const T v0 = (T)(x0 - cx.a0), v1 = (T)(x1 - cx.a1), v2 = (T)(x2 - cx.a2);
                const T wx = tw * tx, wy = tw * ty, wz = tw * tz;
                acc.m[0] += tw;
                acc.m[1] += wx;
                acc.m[2] += wy;
                acc.m[3] += wz;
                acc.m[4] += wx * tx;
                acc.m[5] += wx * ty;
                acc.m[6] += wx * tz;
                acc.m[7] += wy * ty;
                acc.m[8] += wy * tz;
                acc.m[9] += wz * tz;
                acc.r[0] += tw * v0;
                acc.r[1] += tw * v1;
                acc.r[2] += tw * v2;
                acc.r[3] += wx * v0;
                acc.r[4] += wx * v1;
                acc.r[5] += wx * v2;
                acc.r[6] += wy * v0;
                acc.r[7] += wy * v1;
                acc.r[8] += wy * v2;
                acc.r[9] += wz * v0;
                acc.r[10] += wz * v1;
                acc.r[11] += wz * v2;
                acc.g[0] += 1 + ((dx * dx) << 16);
                acc.g[1] += dx + ((dx * dy) << 16);
                acc.g[2] += dy + ((dx * dz) << 16);
                acc.g[3] += dz + ((dy * dy) << 16);
                acc.g[4] += (dy * dz) + ((dz * dz) << 16);
            }
            if (!data) break;
            dx = nx;
            x0 = n0;
            x1 = n1;
            x2 = n2;
            rl = nrl;
        }
    }
}

}  // namespace dev
}  // namespace rmx
