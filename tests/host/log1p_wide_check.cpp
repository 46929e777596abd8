// Host check of kbc::log1p_poly (the wider logarithm polynomials of the exact
// stabilizer) against the C library's log1pl in extended precision, over dense
// grids of their intervals, near zero and at the ends; prints the largest
// relative error of each and fails above the bound given on the command line.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "kbc_device.h"

template <typename C>
static bool check(const char* name, double edge, double bound)
{
    double worst = 0.0, at = 0.0;
    auto one = [&](double x) {
        const long double ref = log1pl((long double)x);
        const double rel = (double)fabsl(((long double)kbc::log1p_poly<C>(x) - ref) / ref);
        if (!(rel <= worst)) { worst = rel; at = x; }
    };
    const int n = 2000000;
    for (int k = -n; k <= n; ++k)
        if (k) one(edge * k / (n + 1.0));
    for (double x = 1e-300; x < edge; x *= 1.37) { one(x); one(-x); }
    one(edge);
    one(-edge);
    std::printf("%s: max relative error %.3e at x = %.17g\n", name, worst, at);
    return worst <= bound;
}

int main(int argc, char** argv)
{
    const double bound = argc > 1 ? std::atof(argv[1]) : 5e-16;
    const bool a = check<kbc::Log1p8>("|x| <= 1/8", 0.125, bound);
    const bool b = check<kbc::Log1p4>("|x| <= 1/4", 0.25, bound);
    return a && b ? 0 : 1;
}
