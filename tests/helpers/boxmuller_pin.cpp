// Largest errors of the Box-Muller functions over all 2^24 arguments each,
// against long double: prints log (ulp), sqrt (ulp), sin and cos (absolute,
// beyond half an ulp of the result), and the largest error of a normal
// relative to max(1, |value|) on a stride of argument pairs, next to the same
// of the C library's functions.
#include "soma_boxmuller.hpp"

#include <math.h>
#include <stdio.h>

using namespace soma;

static double ulp(double v) { return nextafter(fabs(v), INFINITY) - fabs(v); }

int main()
{
    const long double two_pi = 6.283185307179586476925286766559005768L;
    double el = 0, eq = 0, es = 0, ec = 0;
    for (uint32_t k = 0; k < (1u << 24); ++k) {
        const double u = ((double)k + 0.5) * 0x1p-24;
        const double uu[1] = {u};
        double ll[1];
        log_units<1>(uu, ll);
        const double l = ll[0];
        const long double L = logl((long double)u);
        el = fmax(el, (double)(fabsl((long double)l - L) / ulp((double)L)));
        const double z = -2.0 * l, q = sqrt_normal(z);
        const long double Q = sqrtl((long double)z);
        eq = fmax(eq, (double)(fabsl((long double)q - Q) / ulp((double)Q)));
        const double v = (double)k * 0x1p-24;
        double s, c, c2;
        turns(v, v, c, s, c2);
        if (c2 != c) return 1;
        const long double S = sinl(two_pi * (long double)v), C = cosl(two_pi * (long double)v);
        es = fmax(es, (double)fabsl((long double)s - S) - 0.5 * ulp((double)S));
        ec = fmax(ec, (double)fabsl((long double)c - C) - 0.5 * ulp((double)C));
    }
    double mine = 0, lib = 0;
    for (uint32_t k = 0; k < (1u << 24); k += 37) {
        const uint32_t j = (k * 2654435761u) >> 8;
        double xi[3];
        box_muller3(k << 8, j << 8, j << 8, k << 8, xi);
        const double u = ((double)k + 0.5) * 0x1p-24, v = (double)j * 0x1p-24;
        const long double R = sqrtl(-2.0L * logl((long double)u));
        const double r = sqrt(-2.0 * log(u));
        const long double X[2] = {R * cosl(two_pi * v), R * sinl(two_pi * v)};
        const double y[2] = {r * cos(6.283185307179586476925286766559 * v), r * sin(6.283185307179586476925286766559 * v)};
        for (int d = 0; d < 2; ++d) {
            const double n = fmax(1.0, (double)fabsl(X[d]));
            mine = fmax(mine, (double)fabsl((long double)xi[d] - X[d]) / n);
            lib = fmax(lib, (double)fabsl((long double)y[d] - X[d]) / n);
        }
    }
    printf("%.4f %.4f %.3e %.3e %.3e %.3e\n", el, eq, es, ec, mine, lib);
    return 0;
}
