// Host build of the fp64 exponential of the one-pass evaluation, compared with a 113-bit one.
// Prints the largest error in units in the last place: over the normal range, and (of the form that may leave it)
// whether the values at the ends are the expected ones.
#include <quadmath.h>

#include <cmath>
#include <cstdio>
#include <random>

#include "exp64.h"
#include "exp_table.h"

int main() {
    using namespace lantern;
    const unsigned char* tab = reinterpret_cast<const unsigned char*>(EXP_FINE);
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> ref_near(-40.0, 40.0), ref_any(-4096.0, 4096.0), d_near(-40.0, 4.0), d_any(-700.0, 45.0);
    double worst = 0.0;
    long differ = 0;
    for (int i = 0; i < 400000; ++i) {
        const float ref = (float)(i % 3 ? ref_near(rng) : ref_any(rng));
        const float l = (float)(ref + (i % 2 ? d_near(rng) : d_any(rng)));
        const double K = std::rint((double)ref * EXP_UNITS_INV), start = EXP_UNITS_START - K;
        const double v = exp_units((double)l, start, tab);
        const __float128 exact = expq((__float128)l - (__float128)K * M_LN2q / 256);
        int e;
        std::frexp(v, &e);
        const double err = (double)fabsq(((__float128)v - exact) / (__float128)std::ldexp(1.0, e - 53));
        worst = err > worst ? err : worst;
        differ += v != exp_units_any((double)l, start, tab);
    }
    const double start = EXP_UNITS_START;
    const bool ends = exp_units_any(0.0, start, tab) == 1.0 && exp_units_any(-1100.0, start, tab) == 0.0 &&
                      exp_units_any(-5000.0, EXP_UNITS_START + 1400000.0, tab) == 0.0 &&
                      std::fabs(exp_units_any(-720.0, start, tab) / std::exp(-720.0) - 1.0) < 1e-10;
    std::printf("%.6f %ld %d\n", worst, differ, ends ? 1 : 0);
    return 0;
}
