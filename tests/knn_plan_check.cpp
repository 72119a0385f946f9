// Host check of the candidate lists' plan: for every shape of a grid over vocabularies, table widths and codes of
// both types, the selection kernel that plan_pairs() picks is one that the launch has and holds a list of the plan's capacity.
// Prints the shapes whose lists hold keys and tokens; those with keys whose lists exceed 2048 pairs beside 256 candidate
// slots; those with keys of large vocabularies; those with tokens for each of the three kernels; and those that are not held.
#include <cstdio>

#include "knn_plan.h"

int main() {
    const struct { int d, type; } codes[] = {{4, 0}, {8, 0}, {16, 0}, {20, 0}, {8, 1}, {16, 1}, {32, 1}, {256, 1}};
    long keys = 0, tokens = 0, narrow_long = 0, keys_large = 0, kernel[3] = {0, 0, 0}, lost = 0;
    for (const auto& code : codes)
        for (int V = 4096; V <= 1 << 19; V += V / 17 + 1)
            for (int k = 2; k <= 1100; k += 1 + k / 19) {
                const lantern::FilterPlan plan = lantern::filter_plan(V, code.d, k, code.type);
                if (!plan.use) continue;
                const int slots = lantern::candidate_slots(k), pairs = lantern::plan_pairs(plan, k);
                bool built = pairs == 8 || pairs == 12 || pairs == 16;
                if (plan.tokens) {
                    const int vecs = code.d * (code.type == 1 ? 2 : 4) / 16;
                    ++tokens;
                    if (built) ++kernel[pairs / 4 - 2];
                    built = built && slots <= 1024 && (vecs == 1 || vecs == 2 || vecs == 4);
                } else {
                    ++keys;
                    narrow_long += slots <= 256 && plan.cap > 8 * lantern::LIST_THREADS;
                    keys_large += V >= 65536;
                    built = (built && slots <= 1024) || (pairs == 4 && slots <= 256);
                }
                lost += !built || pairs * lantern::LIST_THREADS < plan.cap;
            }
    std::printf("%ld %ld %ld %ld %ld %ld %ld %ld\n", keys, tokens, narrow_long, keys_large, kernel[0], kernel[1], kernel[2], lost);
    return 0;
}
