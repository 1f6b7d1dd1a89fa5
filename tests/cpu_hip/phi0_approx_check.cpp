// The library's phi0 (its device header, built for the host over the HIP emulation) against the
// oracle's, bit for bit, with reciprocals and reciprocal square roots that are as approximate as
// a hardware's: off by up to 2^-BITS of their value, up or down.  The exact ones of the emulation
// would hide a quotient that depends on its seed.  Test infrastructure only.
#include "hip/hip_runtime.h"
#include <cstdio>
#include <cstring>
#include <random>
static int g_bits = 24;
// (the same error for the same operand, as a table's would be)
static inline double off_by(double x, double seed) {
    uint64_t u;
    std::memcpy(&u, &seed, 8);
    u = (u ^ (u >> 31)) * 0x9E3779B97F4A7C15ull;
    u = (u ^ (u >> 29)) * 0xBF58476D1CE4E5B9ull;
    const double e = (double)(int64_t)(u ^ (u >> 32)) / 9223372036854775808.0;   // in [-1, 1)
    return x * (1.0 + std::ldexp(e, -g_bits));
}
static inline double approx_rcp(double x) { return off_by(1.0 / x, x); }
static inline double approx_rsq(double x) { return off_by(1.0 / std::sqrt(x), x); }
#define __builtin_amdgcn_rcp approx_rcp
#define __builtin_amdgcn_rsq approx_rsq
#include "rmx_device.h"
typedef struct { int32_t kind; double centre[3]; double semi[3]; double rot[9]; } orc_shape;
extern "C" double orc_phi0(const orc_shape* s, double x, double y, double z);
int main(int argc, char** argv) {
    const long n = argc > 1 ? atol(argv[1]) : 100000;
    g_bits = argc > 2 ? atoi(argv[2]) : 24;
    std::mt19937_64 g(11);
    std::uniform_real_distribution<double> U(0.0, 1.0);
    std::normal_distribution<double> N(0.0, 1.0);
    long bad = 0;
    for (long i = 0; i < n; ++i) {
        orc_shape o{};
        o.kind = 2;
        for (int a = 0; a < 3; ++a) { o.centre[a] = U(g) - 0.5; o.semi[a] = 0.02 + 0.38 * U(g); }
        if (i % 3 == 0) o.semi[2] *= std::pow(10.0, -4.0 * U(g));             // flat
        if (i % 4 == 0) o.semi[1] = o.semi[0] * (1.0 + (i % 8 ? 1e-15 : 1e-9));
        double q[4]; double qn = 0; for (double& v : q) { v = N(g); qn += v * v; }
        qn = std::sqrt(qn); for (double& v : q) v /= qn;
        const double w = q[0], x = q[1], y = q[2], z = q[3];
        const double R[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                             2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                             2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)};
        for (int k = 0; k < 9; ++k) o.rot[k] = R[k];
        double v[3], dir[3], len = 0.0, at[3];
        for (int a = 0; a < 3; ++a) { dir[a] = N(g); len += dir[a] * dir[a]; }
        // on the surface to rounding, within a few cells of it, or anywhere
        const double off = i % 6 == 0 ? 0.0 : std::pow(10.0, -8.0 * U(g)) * (U(g) < 0.5 ? -1 : 1);
        for (int a = 0; a < 3; ++a) at[a] = dir[a] / std::sqrt(len) * o.semi[a] * (1.0 + off);
        for (int a = 0; a < 3; ++a)
            v[a] = o.centre[a] + (o.rot[3 * a] * at[0] + o.rot[3 * a + 1] * at[1] +
                                  o.rot[3 * a + 2] * at[2]);
        rmx::dev::ShapeR s;
        s.kind = 2;
        s.c0 = o.centre[0]; s.c1 = o.centre[1]; s.c2 = o.centre[2];
        s.e0 = o.semi[0]; s.e1 = o.semi[1]; s.e2 = o.semi[2];
        s.r00 = o.rot[0]; s.r01 = o.rot[1]; s.r02 = o.rot[2];
        s.r10 = o.rot[3]; s.r11 = o.rot[4]; s.r12 = o.rot[5];
        s.r20 = o.rot[6]; s.r21 = o.rot[7]; s.r22 = o.rot[8];
        const double a = rmx::dev::phi0(s, v[0], v[1], v[2]);
        const double b = orc_phi0(&o, v[0], v[1], v[2]);
        if (std::memcmp(&a, &b, 8)) { if (bad < 5) printf("mismatch %.17g %.17g\n", a, b); ++bad; }
    }
    printf("phi0_approx_check: %ld points, %ld mismatches\n", n, bad);
    return bad != 0;
}
