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
    // the form that may leave the normal range, down to 1100 below references of up to 4096 in magnitude
    std::uniform_real_distribution<double> d_low(-1100.0, 45.0);
    double worst_any = 0.0, worst_any_below = 0.0;
    for (int i = 0; i < 400000; ++i) {
        const float ref = (float)(i % 4 == 0 ? -4096.0 : i % 4 == 1 ? 4096.0 : ref_any(rng));
        const float l = (float)(ref + d_low(rng));
        const double K = std::rint((double)ref * EXP_UNITS_INV);
        const double v = exp_units_any((double)l, EXP_UNITS_START - K, tab);
        const __float128 exact = expq((__float128)l - (__float128)K * M_LN2q / 256), err = fabsq((__float128)v - exact);
        if (exact > 0x1p-1021) {
            int e;
            std::frexp(v, &e);
            worst_any = std::fmax(worst_any, (double)(err / (__float128)std::ldexp(1.0, e - 53)));
        } else {
            worst_any_below = std::fmax(worst_any_below, (double)(err / (__float128)std::ldexp(1.0, -1074)));
        }
    }
    // e^d, d <= 0, from the table laid out whole: rounding error where the result is normal, otherwise in units of the
    // smallest number; arguments of any size (what the tree walk subtracts from a maximum near the largest float)
    static uint64_t whole[2 * EXP_FINE_N];
    for (int j = 0; j < EXP_FINE_N; ++j) {
        whole[2 * j] = EXP_FINE[2 * j] + ((uint64_t)j << 44);
        whole[2 * j + 1] = EXP_FINE[2 * j + 1];
    }
    const unsigned char* wtab = reinterpret_cast<const unsigned char*>(whole);
    std::uniform_real_distribution<double> small(-60.0, 0.0), low(-1110.0, 0.0), edge(-746.0, -700.0);
    double worst_nonpos = 0.0, worst_below = 0.0;
    for (int i = 0; i < 400000; ++i) {
        const double d = i % 3 == 0 ? small(rng) : i % 3 == 1 ? low(rng) : edge(rng);
        const double v = exp_units_nonpos(d, wtab);
        const __float128 err = fabsq((__float128)v - expq((__float128)d));
        if (d > -708.0) {
            int e;
            std::frexp(v, &e);
            worst_nonpos = std::fmax(worst_nonpos, (double)(err / (__float128)std::ldexp(1.0, e - 53)));
        } else {
            worst_below = std::fmax(worst_below, (double)(err / (__float128)std::ldexp(1.0, -1074)));
        }
    }
    long wrong = exp_units_nonpos(0.0, wtab) != 1.0;
    for (double d : {-1100.0, -1101.0, -5000.0, -4e10, -1e30, -6.8e38, -1e300, -(double)INFINITY}) wrong += exp_units_nonpos(d, wtab) != 0.0;
    for (double top : {1e6, 3.4e10, 4e10, 1e12, 1e30, -1e30, 3.4e38, -3.4e38})   // a row's maximum, below it nothing or -inf
        for (float l : {(float)top, -3.4028234e38f, -(float)INFINITY})
            wrong += exp_units_nonpos((double)l - (double)(float)top, wtab) !=
                     (l == (float)top || (double)l - (double)(float)top > -700.0 ? std::exp((double)l - (double)(float)top) : 0.0);
    std::printf("%.6f %ld %d %.6f %.6f %ld %.6f %.6f\n", worst, differ, ends ? 1 : 0, worst_nonpos, worst_below, wrong, worst_any,
                worst_any_below);
    return 0;
}
