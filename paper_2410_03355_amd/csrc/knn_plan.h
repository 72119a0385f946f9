// Plan of the neighbour table's sampled-threshold path (host code): for a shape, the sample, the rank of the
// threshold in it and the capacity of a row's candidate list; for a plan, the selection kernel that holds it.
#pragma once

#include <math.h>

namespace lantern {

// Tails of the binomial law of n trials with success probability p, summed term by term from the
// given end (the terms fall off geometrically there): P(X >= r) and P(X <= r).
inline double binomial_log_pmf(int n, double p, int x) {
    return lgamma((double)n + 1.0) - lgamma((double)x + 1.0) - lgamma((double)(n - x) + 1.0) + (double)x * log(p) +
           (double)(n - x) * log1p(-p);
}
inline double binomial_upper_tail(int n, double p, int r) {
    if (r <= 0) return 1.0;
    if (r > n) return 0.0;
    double term = exp(binomial_log_pmf(n, p, r)), sum = 0.0;
    for (int x = r; x <= n && (term > 1e-300 || x < (int)(n * p)); ++x) {
        sum += term;
        term *= (double)(n - x) / (double)(x + 1) * p / (1.0 - p);
        if (x > (int)(n * p) && term < sum * 1e-17) break;
    }
    return sum;
}
inline double binomial_lower_tail(int n, double p, int r) {
    if (r < 0) return 0.0;
    if (r >= n) return 1.0;
    double term = exp(binomial_log_pmf(n, p, r)), sum = 0.0;
    for (int x = r; x >= 0; --x) {
        sum += term;
        if (x == 0) break;
        term *= (double)x / (double)(n - x + 1) * (1.0 - p) / p;
        if (x < (int)(n * p) && term < sum * 1e-17) break;
    }
    return sum;
}

// Plan of the sampled-threshold path for one shape.  A row's threshold has between `rank` and
// `rank + slack` of the row's keys to `S` sampled tokens at or below it.  The row's list is too short
// (fewer than the k-1+pad candidates the selection wants) only if at least rank - 1 of the sampled
// tokens are among the row's k-2+pad nearest, and too long for its `cap` slots only if at most
// rank + slack of them are among its cap+1 nearest (the row's own token may be in the sample: hence
// the - 1).  The sample takes one token from each of S strata of the vocabulary, so the number of
// sampled tokens in a given set is a sum of independent trials, whose tails are no heavier than
// those of the binomial law with the same mean (Hoeffding): `rank` is the smallest and `cap` the
// smallest of 1024 .. 4096 for which that bound puts either miss below 1e-10 per row, whatever
// the codebook.  A row that misses all the same is flagged and ranked by the all-pairs pass.
// use == false: the shape takes the whole-key-block path.
struct FilterPlan {
    bool use;
    bool tokens;   // the lists hold tokens alone and every listed one's key is evaluated in fp64
    bool wide_tiles;   // (tokens) 512 tokens to a tile of the filtering contraction instead of 128
    int S;      // sampled tokens, a multiple of 64, at most 4096
    int rank;   // the threshold has between rank and rank + slack of a row's S sample keys at or below it
    int slack;
    int cap;    // slots of a row's candidate list: 1024, 2048, 3072 or 4096
};

// Candidates wanted of a row: its k - 1 others and a few more, so that the proof that none is missing passes.
inline int candidate_slots(int k) { return (k - 1) + 8 + (k - 1) / 128; }

constexpr int FILTER_STAGE = 8192;   // hits of a tile that are staged at once

inline double normal_density(double z) { return exp(-0.5 * z * z) * 0.39894228040143267794; }
// z with P(X > z) = share of a standard normal, by halving (0 < share < 1; to 1e-6, a first guess is made of it).
inline double normal_upper_quantile(double share) {
    double lo = -8.0, hi = 8.0;
    for (int i = 0; i < 24; ++i) {
        const double mid = 0.5 * (lo + hi);
        (0.5 * erfc(mid * 0.70710678118654752440) > share ? lo : hi) = mid;
    }
    return 0.5 * (lo + hi);
}

inline FilterPlan filter_plan(int V, int d, int k, int cb_dtype) {
    FilterPlan P = {false, false, false, 0, 0, 0, 0};
    const bool vec = cb_dtype == 1 ? (d % 8) == 0 : (d % 4) == 0;   // what the matrix-core kernels need
    const int want = candidate_slots(k);
    // 64 candidates or fewer: the lists would be several times longer than what the selection wants
    if (!vec || V < 4096 || want <= 64 || want > 1024) return P;
    int S = V / 8;
    if (S > 4096) S = 4096;
    S = S / 64 * 64;
    const double miss = 1e-10;
    const double others = (double)(V - 1);
    // too short: Binomial(S, (want - 1) / (V - 1)) >= rank - 1
    const double p_lo = (double)(want - 1) / others;
    int rank = (int)(S * p_lo) + 2;
    while (rank < S && binomial_upper_tail(S, p_lo, rank - 1) > miss) ++rank;
    if (rank >= S) return P;
    // the search for the threshold stops anywhere between rank and rank + slack (a sixteenth more)
    const int slack = rank / 16 < S - rank ? rank / 16 : S - rank;
    // too long: Binomial(S, (cap + 1) / (V - 1)) <= rank + slack
    int cap = 0;
    for (int c = 1024; c <= 4096 && cap == 0; c += 1024) {
        const double p_hi = (double)(c + 1) / others;
        if (p_hi >= 1.0 || binomial_lower_tail(S, p_hi, rank + slack) <= miss) cap = c;
    }
    if (cap == 0) return P;
    P.use = true;
    // A list without keys costs the selection the exact keys of all it holds instead of `want` of them, and saves the
    // keys' way through memory and the phases that narrow the list.  It pays where codes are short, and the
    // lists are not much longer than what is wanted of them or the contraction over a large vocabulary outweighs the
    // selection.  Whole builds, pairs / tokens: codes of 32 bytes, V = 4096, k = 64 (surplus 3.2) 50 / 55 us, k = 1000
    // 104 / 91; V = 6500, k = 100 75 / 79, k = 500 107 / 96; V = 8192, k = 200 105 / 98; V = 16384, k = 1000 355 / 292;
    // V = 60000, k = 230 2772 / 1809.  Codes of 64 bytes: V = 8192, k = 100 104 / 113, k = 1000 167 / 172; V = 12288,
    // k = 300 199 / 191, k = 1000 (cosine) 296 / 377; V = 16384, k = 300 (cosine) 328 / 298; V = 33000, k = 100 994 / 807.
    const double listed = (rank + 0.5 * slack) / S * V;
    const int row_bytes = d * (cb_dtype == 1 ? 2 : 4);
    if (row_bytes == 16 || row_bytes == 32) P.tokens = V >= 8192 || listed <= 2.0 * want;
    else if (row_bytes == 64) P.tokens = V >= 12288 && listed <= 1024;
    // Four times the tokens to a reservation of list slots, as long as their hits are staged at once and there are
    // tiles for every compute unit several times over.
    P.wide_tiles = listed / V * (128.0 * 512.0) <= 0.85 * FILTER_STAGE && V >= 8192;
    P.S = S;
    P.rank = rank;
    P.slack = slack;
    P.cap = cap;
    return P;
}

// The selection holds a row's list in registers, on LIST_THREADS threads per row: pairs per thread, one of
// 4, 8, 12 or 16 (4 only with 256 candidate slots; the other size is 1024), such that pairs times threads is
// at least `cap` and a list of up to cap pairs is held whole.  Narrow tables of large vocabularies have long
// lists too (V = 131072, k = 100: cap 3072).
constexpr int LIST_THREADS = 256;
inline int list_pairs(int candidate_slots, int cap) {
    const int least = candidate_slots <= 256 ? 4 : 8;
    const int pairs = (cap + LIST_THREADS * 4 - 1) / (LIST_THREADS * 4) * 4;
    return pairs < least ? least : pairs;
}
// What a plan's selection holds per thread: lists of tokens have 1024 candidate slots whatever is wanted of them.
inline int plan_pairs(const FilterPlan& plan, int k) { return list_pairs(plan.tokens ? 1024 : candidate_slots(k), plan.cap); }

}  // namespace lantern
