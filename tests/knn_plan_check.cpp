// Host check of the candidate lists' plan: for every shape of a grid over vocabularies and table widths, the
// selection kernel that list_pairs() picks holds a list of the plan's capacity.  Prints the shapes that use
// the path, those whose lists exceed 2048 pairs beside 256 candidate slots, and those that are not held.
#include <cstdio>

#include "knn_plan.h"

int main() {
    long used = 0, narrow_long = 0, lost = 0;
    for (int V = 4096; V <= 1 << 19; V += V / 23 + 1)
        for (int k = 2; k <= 1100; k += 1 + k / 29) {
            const lantern::FilterPlan plan = lantern::filter_plan(V, 8, k, 0);
            if (!plan.use) continue;
            ++used;
            const int slots = (k - 1) + 8 + (k - 1) / 128;
            const int pairs = lantern::list_pairs(slots, plan.cap);
            const bool built = (pairs == 4 && slots <= 256) || pairs == 8 || pairs == 12 || pairs == 16;
            narrow_long += slots <= 256 && plan.cap > 8 * lantern::LIST_THREADS;
            lost += !built || pairs * lantern::LIST_THREADS < plan.cap;
        }
    std::printf("%ld %ld %ld\n", used, narrow_long, lost);
    return 0;
}
