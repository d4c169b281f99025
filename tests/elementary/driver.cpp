// log_d, log1p_d and quotient_d of the kernels, compiled for the host (the seed of the reciprocal is worse here than the device's),
// against long double.  Prints the largest error in units of the last place per range, then the special values.
#include <algorithm>
#include <cstdio>
#include <random>

#include "elementary.h"

static double ulps(double got, long double ref) {
    int e;
    std::frexp((double)ref, &e);
    return (double)(fabsl((long double)got - ref) / ldexpl(1.0L, e - 53));
}

int main() {
    std::mt19937_64 gen(7);
    std::uniform_real_distribution<double> unit(0.0, 1.0);
    struct Range { bool plus_one, logarithmic; double lo, hi; };
    const Range ranges[] = {{false, false, 0.5, 2.0},  {false, false, 0.999, 1.001}, {false, true, 1e-300, 1e300}, {false, true, 1e-320, 1e-300},
                            {true, false, -0.5, 1.0},  {true, false, -0.999999, -0.4}, {true, true, 1e-25, 1.0},   {true, true, 1e-2, 1e200},
                            {true, true, 1e-16, 1e-6}, {true, true, -1e-16, -1e-6}};
    for (const Range& r : ranges) {
        double worst = 0.0;
        for (int i = 0; i < 400000; ++i) {
            const double t = unit(gen);
            const double sign = r.logarithmic && r.lo < 0.0 ? -1.0 : 1.0;
            const double x = r.logarithmic ? sign * std::exp(std::log(sign * r.lo) + t * (std::log(sign * r.hi) - std::log(sign * r.lo)))
                                           : r.lo + t * (r.hi - r.lo);
            const double err = r.plus_one ? ulps(lb::log1p_d(x), log1pl((long double)x)) : ulps(lb::log_d(x), logl((long double)x));
            if (!(err <= worst)) worst = err;
        }
        std::printf("range %s %g %g %.6f\n", r.plus_one ? "log1p" : "log", r.lo, r.hi, worst);
    }
    double worst = 0.0;
    for (int i = 0; i < 400000; ++i) {
        const double e = std::exp(-700.0 * unit(gen) * unit(gen)), z = 1.0 + e, a = i & 1 ? 1.0 : e;
        worst = std::max(worst, ulps(lb::quotient_d(a, z), (long double)a / (long double)z));
    }
    std::printf("quotient %.6f\n", worst);
    const double special[] = {0.0, INFINITY, -INFINITY, NAN, -1.0, -2.0, 1.0, 5e-324, 1.7976931348623157e308};
    for (double x : special) std::printf("at %.17g %.17g %.17g %.17g %.17g\n", x, lb::log_d(x), std::log(x), lb::log1p_d(x), std::log1p(x));
    return 0;
}
