// Host build of the short exponential for non-positive arguments, compared with the general one.
#include <cmath>
#include <cstdio>
#include <random>

#include "exp64.h"
#include "exp_table.h"

int main() {
    std::mt19937_64 rng(11ull);
    std::uniform_real_distribution<double> near(-60.0, 0.0), far(-1100.0, 0.0);
    long differ = 0;
    for (int i = 0; i < 2000000; ++i) {
        double d = (i & 1) ? near(rng) : far(rng);
        if (i % 3 == 0) d = (double)(float)d;
        differ += lantern::exp_tab_nonpos(d, lantern::EXP_TABLE_HILO) != lantern::exp_tab(d, lantern::EXP_TABLE_HILO);
    }
    const double edges[] = {0.0, -0.0, -700.0, -708.4, -745.1, -746.0, -1000.0, -1e300, -INFINITY};
    for (double d : edges)
        differ += lantern::exp_tab_nonpos(d, lantern::EXP_TABLE_HILO) != lantern::exp_tab(d, lantern::EXP_TABLE_HILO);
    std::printf("%ld\n", differ);
    return 0;
}
