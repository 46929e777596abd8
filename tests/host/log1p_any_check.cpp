// Host check of kbc::log1p_any (the exact stabilizer's logarithm away from
// equilibrium) against the C library's log1pl in extended precision: towards -1, both
// sides of the mantissa split and of powers of two, near zero and far above one;
// prints the largest error over 1 + |ln(1 + x)| and fails above the bound given
// on the command line.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "kbc_device.h"

int main(int argc, char** argv)
{
    const double bound = argc > 1 ? std::atof(argv[1]) : 3e-16;
    double worst = 0.0, at = 0.0;
    auto one = [&](double x) {
        if (!(x > -1.0)) return;
        const long double ref = log1pl((long double)x);
        const double e = (double)(fabsl((long double)kbc::log1p_any(x) - ref) / (1.0L + fabsl(ref)));
        if (!(e <= worst)) { worst = e; at = x; }
    };
    const int n = 1000000;
    for (int k = 1; k <= n; ++k) one(-1.0 + 4.0 * k / n);        // (-1, 3]
    for (double d = 0x1p-53; d < 1.0; d *= 1.003) one(-1.0 + d);   // towards -1
    for (double x = 1e-300; x < 1e300; x *= 1.01) { one(x); one(-x); }
    for (int k = -50; k < 60; ++k)
        for (double m : {1.0, 0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp+0}) {
            const double v = std::ldexp(m, k), x = v - 1.0;
            for (double y : {x, std::nextafter(x, -1.0), std::nextafter(x, 1e300)}) one(y);
        }
    one(0.0);
    std::printf("largest error %.3e of 1 + |ln(1 + x)| at x = %.17g\n", worst, at);
    return worst <= bound ? 0 : 1;
}
