// soma_boxmuller.hpp -- FP64 Box-Muller on 24-bit uniforms.
//
// The normals of the bond-force-biased moves take logarithms, roots, sines and
// cosines of numbers that are known to be k 2^-24 (or (k + 1/2) 2^-24) in
// (0, 1): no zeros, infinities, subnormals or large angles.  The functions
// here use that; the three normals of a bead take 140 vector instructions
// where the device library's general functions take about 500 (96 for a
// logarithm, 20 for a root, 90 for a sine or cosine), and the sweep with such
// moves is bound by vector issue (1514 instructions per wave with those): 4.2M
// beads take 61.6 us per sweep, 89 with the library's functions.
//
//   logarithm  u = 2^e m, m in [1/sqrt(2), sqrt(2)), f = m - 1, s = f / (2 + f):
//              ln m = 2 artanh s = f - s (f - s^2 Q(s^2)), Q = 2/3 + 2/5 s^2 + ...
//              as a polynomial of seven terms (remainder 2^-56.6 of s),
//              ln 2 in two parts.
//   cosine     w = |u - 1/2|: cos 2 pi u = sin 2 pi (w - 1/4), the new angle
//   and sine   exact and within a quarter turn; sin 2 pi u the same of
//              1/4 - |w - 1/4|, with the sign of 1/2 - u.  One polynomial in the
//              square (eight terms and 2 pi in two parts, remainder 2^-55.7 of
//              the leading term) serves all three, so its coefficients are
//              loaded once; with an octant reduction the sine and the cosine
//              each want their own.  No rounding of the angle 2 pi u, which
//              alone costs up to 4.4e-16.
//   root       one reciprocal-root estimate, Goldschmidt steps, one residual.
//
// The polynomials interpolate the series at the Chebyshev nodes of the range,
// their coefficients rounded to nearest.
//
// Largest errors over every one of the 2^24 arguments (CPU, long double):
// logarithm 0.88 ulp, root 0.50 ulp, sine and cosine 1.9e-16 beyond half an ulp
// of the result; a normal is within 4.0e-16 of its value (relative to
// max(1, |value|)), with the C library's functions of the rounded angle 2.5e-15.
//
// Host builds (tests) take the estimates from FP32 division and root.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>

#if defined(__HIPCC__)
#define SOMA_HD __host__ __device__ __forceinline__
#else
#define SOMA_HD static inline
#endif

namespace soma {

SOMA_HD double rcp_estimate(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcp(x);
#else
    return (double)(1.0f / (float)x);
#endif
}
SOMA_HD double rsq_estimate(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rsq(x);
#else
    return (double)(1.0f / sqrtf((float)x));
#endif
}

// ln u[i] for u[i] in [2^-25, 1).
template <int N>
SOMA_HD void log_units(const double (&u)[N], double (&l)[N])
{
    double f[N], s[N], z[N], q[N], ed[N];
    for (int i = 0; i < N; ++i) {
        // exponent and mantissa: adding the distance of 1/sqrt(2) to 1 in the
        // high word puts m into [1/sqrt(2), sqrt(2))
        uint64_t b;
        memcpy(&b, &u[i], sizeof b);
        const uint32_t hi = (uint32_t)(b >> 32) + (0x3FF00000u - 0x3FE6A09Eu);
        ed[i] = (double)((int)(hi >> 20) - 1023);
        b = (uint64_t)((hi & 0x000FFFFFu) + 0x3FE6A09Eu) << 32 | (uint32_t)b;
        double m;
        memcpy(&m, &b, sizeof m);
        f[i] = m - 1.0;
        // s = f / (2 + f)
        const double d = 2.0 + f[i];
        double r = rcp_estimate(d);
        r = fma(fma(-d, r, 1.0), r, r);
        r = fma(fma(-d, r, 1.0), r, r);
        s[i] = f[i] * r;
        s[i] = fma(fma(-d, s[i], f[i]), r, s[i]);
        z[i] = s[i] * s[i];
    }
    const double k0 = 0x1.2b5f68a50d903p-3, k1 = 0x1.39fdcceb4bb45p-3, k2 = 0x1.7462b91b8df65p-3,
                 k3 = 0x1.c71c62d5e53e0p-3, k4 = 0x1.2492492dfd86cp-2, k5 = 0x1.9999999995273p-2,
                 k6 = 0x1.5555555555558p-1;
    for (int i = 0; i < N; ++i) q[i] = fma(k0, z[i], k1);
    for (int i = 0; i < N; ++i) q[i] = fma(q[i], z[i], k2);
    for (int i = 0; i < N; ++i) q[i] = fma(q[i], z[i], k3);
    for (int i = 0; i < N; ++i) q[i] = fma(q[i], z[i], k4);
    for (int i = 0; i < N; ++i) q[i] = fma(q[i], z[i], k5);
    for (int i = 0; i < N; ++i) q[i] = fma(q[i], z[i], k6);
    // ln 2 = hi + lo, hi with 33 bits: e hi is exact
    const double ln2_hi = 0x1.62e42fefp-1, ln2_lo = 0x1.473de6af278edp-34;
    for (int i = 0; i < N; ++i) {
        const double tail = fma(ed[i], ln2_lo, -(s[i] * fma(-z[i], q[i], f[i])));
        l[i] = fma(ed[i], ln2_hi, f[i] + tail);
    }
}

// sqrt z for z well inside the normal range.
SOMA_HD double sqrt_normal(double z)
{
    const double y = rsq_estimate(z);
    double g = z * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, z), h, g);
}

// sin 2 pi r[i] for |r[i]| <= 1/4 (r^2 exact: r has at most 24 bits).
template <int N>
SOMA_HD void sin_turns(const double (&r)[N], double (&v)[N])
{
    const double k0 = 0x1.9ec5cdbeecd34p-4, k1 = -0x1.6f866b70b27bdp-1, k2 = 0x1.e8f3b0121aafdp+1,
                 k3 = -0x1.e3074ee5f4a61p+3, k4 = 0x1.50783486f190cp+5, k5 = -0x1.32d2cce62adb9p+6,
                 k6 = 0x1.466bc6775aad6p+6, k7 = -0x1.4abbce625be53p+5;
    const double two_pi_hi = 0x1.921fb54442d18p+2, two_pi_lo = 0x1.1a62633145c07p-52;
    double x[N], p[N];
    for (int i = 0; i < N; ++i) x[i] = r[i] * r[i];
    for (int i = 0; i < N; ++i) p[i] = fma(k0, x[i], k1);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k2);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k3);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k4);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k5);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k6);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], k7);
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], two_pi_lo);
    for (int i = 0; i < N; ++i) v[i] = fma(r[i], two_pi_hi, r[i] * p[i]);
}

// cos 2 pi u, sin 2 pi u and cos 2 pi t for u, t in [0, 1).
SOMA_HD void turns(double u, double t, double &cu, double &su, double &ct)
{
    const double w = 0.5 - u, qc = fabs(w) - 0.25;
    const double r[3] = {qc, copysign(0.25 - fabs(qc), w), fabs(t - 0.5) - 0.25};
    double v[3];
    sin_turns<3>(r, v);
    cu = v[0];
    su = v[1];
    ct = v[2];
}

// Three standard normals from the four words of a Philox block: words 0, 1
// give the first two, words 2, 3 the third.
SOMA_HD void box_muller3(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, double xi[3])
{
    const double u[2] = {((double)(w0 >> 8) + 0.5) * 0x1p-24, ((double)(w2 >> 8) + 0.5) * 0x1p-24};
    double l[2], cu, su, ct;
    log_units<2>(u, l);
    const double r1 = sqrt_normal(-2.0 * l[0]), r2 = sqrt_normal(-2.0 * l[1]);
    turns((double)(w1 >> 8) * 0x1p-24, (double)(w3 >> 8) * 0x1p-24, cu, su, ct);
    xi[0] = r1 * cu;
    xi[1] = r1 * su;
    xi[2] = r2 * ct;
}

}  // namespace soma
