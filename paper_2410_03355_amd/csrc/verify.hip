// Relaxed-acceptance verification (Section 4.3; Algorithm 2, inference part;
// Algorithm 1, accept / resample branch) for gfx950.
//
// One workgroup per row, two code paths inside the same launch:
//   fast path   fp32.  Streams the target and draft rows from HBM once with
//               16-byte loads, keeps the raw target row in LDS, gathers the
//               draft token's k neighbours from LDS, prefix-scans them and
//               takes the TVD cut and the acceptance test.  Each comparison
//               carries a rounding margin; a row is settled here only when
//               every comparison it took cleared its margin and it is accepted
//               (or, when only decisions are asked for, definitely rejected).
//   exact path  fp64.  The workgroup of a row the fast path did not settle
//               (ambiguous comparison, unusable input, a rejected row whose
//               resampled token is wanted) re-evaluates it: same rule, then
//               the residual and its inverse CDF.
// The fast path takes any row of 16 bytes up to 128 KiB, at any address: 256, 512 or
// 1024 threads per row.  Other shapes (and diagnostics of rows that are not 16-byte
// aligned whole vectors) run the exact path for every row (kernel verify_exact).
// Three modes (verify_args.h): decisions and resampled tokens; decisions only;
// the fp64 path for selected verifications in 512-thread workgroups
// (resample_selected, and tree_finish, which first walks its draft tree; draw_from_registers
// says which plain tree steps end in the kernel of sequential.hip instead).
// Letters: t = target probability (the paper's q), g = drafter probability
// (the paper's p), xt = draft token.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stddef.h>
#include <math.h>
#include <stdint.h>

#include "exp_table.h"
#include "fast_cut.h"
#include "lds_limit.h"
#include "sequential_args.h"
#include "tree_walk.h"
#include "verify_args.h"
#include "verify_common.h"

namespace lantern {

// LDS layout of verify_fast after the raw row
template <int TNW>
struct FastShared {
    float wmax_t[TNW], wmax_g[TNW]; // per-wave maxima over the sampled part of the row
    float wsum_t[TNW], wsum_g[TNW]; // per-wave sums of exponentials
    float wtot[TNW];                // per-wave totals of the neighbour terms (first four slots per thread)
    int wbad[TNW];                  // a table entry outside [0,V)
    int cut_np[TNW];                // per wavefront: first slot not definitely inside the bound,
    int cut_df[TNW];                //   first slot definitely outside it,
    float cut_s[TNW];               //   sum before the former
    int tail[4];                    // longer table rows: the result of the walk beyond those slots (a_size, S, definite, bad)
};                                  // followed by the exact path's region
static_assert(sizeof(FastShared<4>) % 16 == 0 && sizeof(FastShared<8>) % 16 == 0 && sizeof(FastShared<16>) % 16 == 0,
              "the exact path's LDS region must be 16-byte aligned");

template <typename LT, int FORM, int TNT = NT>
__device__ __forceinline__ void exact_row(const VerifyArgs& a, int row, unsigned char* ex, const unsigned char* lds_row,
                          bool have_max, float max_t, float max_g, const unsigned char* lds_grow = nullptr,
                          unsigned char* tab_lds = nullptr);

// What a kernel of the fp32 pass knows about its rows.
//   ROWS_FULL   16-byte aligned, and every vector slot of every thread is filled: no bounds checks
//   ROWS_WHOLE  16-byte aligned whole vectors, not every slot filled: slots beyond the row are not loaded
//   ROWS_ANY    any address and any length of at least one vector: every slot is loaded, clamped to the row
enum RowsKnown { ROWS_FULL, ROWS_WHOLE, ROWS_ANY };

// ---------------------------------------------------------------------------
// fp64 evaluation of a row in one pass, with what the fp32 pass already knows
// ---------------------------------------------------------------------------
// For a row the fp32 pass could not settle but found usable, with both sums in range and a
// definite cut: the decision and, on rejection, the resampled token, in fp64, in ONE pass over the
// two rows (2V exponentials instead of the 4V of the general path, no pass for the maxima).
// What makes one pass enough: the residual max(0, t_A - g) needs, token by token, the SIGN of
// t_A(x) - g(x), and the fp32 terms and sums decide that sign for all but the few tokens where
// the two probabilities agree to within the fp32 error bound.  So while the pass adds up the
// fp64 normalisers it also adds, per (vector chunk, wavefront) segment and in token order, the
// target and drafter terms of the tokens whose residual is certainly positive; tokens whose sign
// fp32 cannot tell go on a short list with their fp64 terms.  Once the normalisers are known a
// segment's residual mass is  P_t / Z_t - P_g / Z_g  plus its listed tokens, a scan over the
// segment masses (one per vector slot and wavefront: up to 128 with 1024 threads) finds the segment
// that holds the draw, and that segment alone is re-evaluated token by token.
// Bound by the issue of vector instructions: 43 a token, 15 of them for each exponential (exp_units), against 80 with
// A looked up in a bit mask, a reference subtracted from every logit, registers moved down for every two tokens and a
// wavefront sum for every vector.  3840 rows of 16384 bf16 logits of which 45 % are rejected: 125 -> 102 us, of 8192
// fp32 logits 82 -> 63; 960 rows of 8192 bf16 at any address 35 -> 27, of 65536 bf16 234 -> 182.
// No global load sits inside the pass (under a saturated memory system each costs microseconds):
// the drafter's row is fetched again, all of it at once, before the pass starts (keeping it in
// registers from the fp32 pass on would cost that pass registers it does not have), the target row
// is in LDS, the first four table slots per thread in registers.
constexpr int AMB_CAP = 40;          // tokens whose residual sign fp32 leaves open (about one per row)
constexpr double TAU_SIGN = 2.0e-5;  // covers the error of ln(Z_t32 / Z_g32) in the sign test (<= 8.8e-6)

struct AmbEntry {
    double et, eg;   // unnormalised fp64 terms
    int x;           // token
    int pad;
};

// LDS of this path, behind the row and the reductions (the general path's data take the same region).
struct OnePassLayout {
    size_t seg, keep, amb_count, amb, total;
};
// The exponential's table is an LDS object of its own beside the dynamic part.  The general path, which comes after this
// one or instead of it, keeps its own (smaller) table there.
constexpr int EXP_TABLE_BYTES = 2 * EXP_TABLE_N * (int)sizeof(double);
constexpr int EXP_FINE_BYTES = 2 * EXP_FINE_N * (int)sizeof(double);
__host__ __device__ inline OnePassLayout one_pass_layout(int segments) {
    OnePassLayout L;
    size_t off = (sizeof(ExactShared) + 15) & ~size_t(15);
    L.seg = off;       off += (size_t)segments * 2 * sizeof(double);
    L.keep = off;      off += 4 * sizeof(double);
    L.amb = off;       off += AMB_CAP * sizeof(AmbEntry);
    L.amb_count = off; off += 16;
    L.total = off;
    return L;
}

// max of two floats, the second uniform, as the one hardware instruction (fmaxf first quiets both operands, two more
// instructions per call; no NaN reaches this path).
__device__ __forceinline__ float max_f32_1(float a, float uniform) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "s"(uniform), "v"(a));
    return r;
}
// A row's terms e^l 2^(-K/256), K its reference logit in steps of ln2/256.  floor: the least logit that is
// evaluated as it is; lower ones (filtered tokens at -inf among them) are evaluated there.  The target's floor lies
// 700 below its reference and the drafter's 650: terms of 1e-282 of the sum at most, and a target logit at its floor
// is below any drafter logit by more than the sums can make up for (both lie in [1, 2^46]).  What such terms decide is the
// sign of a residual below 1e-260 of the row, which a draw above zero never reaches.
struct UnitRow {
    double start;    // EXP_UNITS_START - K
    float floor;
    __device__ __forceinline__ double arg(float l) const { return (double)max_f32_1(l, floor); }
    __device__ __forceinline__ double term(float l, const unsigned char* tab) const { return exp_units(arg(l), start, tab); }
    // a single term that a decision looks at: nothing at -inf
    __device__ __forceinline__ double term_any(float l, const unsigned char* tab) const {
        return exp_units_any((double)fmaxf(l, floor - 400.f), start, tab);
    }
};
constexpr float UNITS_MAX_REF = 4096.f;      // what exp_units allows, floors and terms above the reference included
__device__ __forceinline__ UnitRow unit_row(float ref, float below) {
    UnitRow r;
    r.start = EXP_UNITS_START - __builtin_rint((double)ref * EXP_UNITS_INV);
    r.floor = uniform_f(ref - below);
    return r;
}

// What the pass does for the EPV tokens of a vector: their fp64 terms into the normalisers, and into the segment's
// sums when the residual is certainly positive; returns whether some token of the lane is neither that nor
// certainly without residual.
// The sign test works on the logits: t(x) > g(x) <=> l_t - l_g > ln(Z_t / Z_g) + r_t - r_g, where only the two
// fp32 sums carry an error (at most 4.4e-6 relative each: terms 2.5e-6, tree sums 1.9e-6, i.e. 8.8e-6 on the
// logarithm), so a margin of TAU_SIGN = 2e-5 on either side makes "positive" and "not positive" certain.
struct OnePassAcc {
    double zt, zg;
};
typedef uint32_t u2x32 __attribute__((ext_vector_type(2)));
template <typename LT>
__device__ __forceinline__ bool one_pass_vector(const uint4& tv, const uint4& gv, const UnitRow& rt, const UnitRow& rg,
                                                double sign_hi, double sign_lo, const unsigned char* tab,
                                                OnePassAcc& acc, double* pt, double* pg) {
    using L = Lane<LT>;
    bool open = false;
    double st = 0.0, sg = 0.0;
#pragma unroll
    for (int e = 0; e < L::EPV; ++e) {
        const double at = rt.arg(L::get(tv, e)), ag = rg.arg(L::get(gv, e));
        const double et = exp_units(at, rt.start, tab);
        const double eg = exp_units(ag, rg.start, tab);
        const double dd = at - ag;
        const bool pos = dd > sign_hi;
        open |= (dd > sign_lo) & !pos;
        acc.zt += et;
        acc.zg += eg;
        const double one = pos ? 1.0 : 0.0;
        st = __builtin_fma(et, one, st);
        sg = __builtin_fma(eg, one, sg);
        // the sums so far are due here: left alone, the compiler keeps the terms of all tokens in registers it lacks
        if (e % 2 == 1) asm volatile("" : "+v"(acc.zt), "+v"(acc.zg), "+v"(st), "+v"(sg));
    }
    *pt = st;
    *pg = sg;
    return open;
}

// Sums over the wavefront of N pairs of doubles per lane, v[2 i] and v[2 i + 1]: out(i, which, sum) is run by
// one lane for each.  Two values to a register at each of the first two steps (halves of the wavefront, then rows of 16
// lanes, exchanged between two registers), so that N = 8 pairs take 72 instructions; one scan each would be 320.
__device__ __forceinline__ double fold_halves(double a, double b) {   // lanes 0..31: a's sum, 32..63: b's
    u2x32 lo = __builtin_bit_cast(u2x32, a), hi = __builtin_bit_cast(u2x32, b);
    const auto x = __builtin_amdgcn_permlane32_swap(lo[0], hi[0], false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(lo[1], hi[1], false, false);
    return __builtin_bit_cast(double, u2x32{x[0], y[0]}) + __builtin_bit_cast(double, u2x32{x[1], y[1]});
}
__device__ __forceinline__ double fold_rows(double a, double b) {     // rows 0, 2 of 16 lanes: a's, rows 1, 3: b's
    u2x32 lo = __builtin_bit_cast(u2x32, a), hi = __builtin_bit_cast(u2x32, b);
    const auto x = __builtin_amdgcn_permlane16_swap(lo[0], hi[0], false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(lo[1], hi[1], false, false);
    return __builtin_bit_cast(double, u2x32{x[0], y[0]}) + __builtin_bit_cast(double, u2x32{x[1], y[1]});
}
template <int N, typename F>
__device__ __forceinline__ void wave_pair_sums(const double (&v)[2 * N], int lane, F out) {
    double w[N];
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = fold_halves(v[2 * i], v[2 * i + 1]);
    if constexpr (N == 1) {
        double s = w[0];
        s += dpp_d<DPP_ROW_SHR1, 0xF>(s);
        s += dpp_d<DPP_ROW_SHR2, 0xF>(s);
        s += dpp_d<DPP_ROW_SHR4, 0xF>(s);
        s += dpp_d<DPP_ROW_SHR8, 0xF>(s);
        s += dpp_d<DPP_ROW_BCAST15, 0xA>(s);
        if ((lane & 31) == 31) out(0, lane >> 5, s);
    } else {
#pragma unroll
        for (int i = 0; i < N; i += 2) {
            double s = fold_rows(w[i], w[i + 1]);
            s += dpp_d<DPP_ROW_SHR1, 0xF>(s);
            s += dpp_d<DPP_ROW_SHR2, 0xF>(s);
            s += dpp_d<DPP_ROW_SHR4, 0xF>(s);
            s += dpp_d<DPP_ROW_SHR8, 0xF>(s);
            if ((lane & 15) == 15) out(i + ((lane >> 4) & 1), lane >> 5, s);
        }
    }
}

// s_row: raw target row in LDS.
// nb: table slots 4*tid .. 4*tid+3.  ref_t, ref_g: the fp32 pass's reference logits; Zt32, Zg32:
// its sums; a_size: its (definite) cut.
// tab_lds: where the exponential's table goes.
// Returns false (the same in every thread) when the row is left to the general path.
template <typename LT, int TNT, int NV, int ROWS>
__device__ __forceinline__ bool exact_one_pass(const VerifyArgs& a, int row, int lrow,
                                               const int (&nb)[4], float ref_t, float ref_g,
                                               float Zt32, float Zg32, int a_size, int xt, float lg_tok, float u_acc32,
                                               unsigned char* tab_lds, unsigned char* ex,
                                               unsigned char* s_row) {
    using L = Lane<LT>;
    constexpr int EPV = L::EPV;
    constexpr int TNW = TNT / WAVE;
    constexpr bool FULL = ROWS == ROWS_FULL;
    constexpr int NSEG = NV * TNW;                           // one wavefront scans them, 64 at a time
    int tid = threadIdx.x;
    // Workgroups of 1024 threads have no registers to keep the drafter's addresses in from the fp32 pass on: stored to
    // scratch memory between that pass's loads they hold up every row, rejected or not (decisions of 960 rows of 40000
    // bf16 logits 56.2 -> 53.2 us, and the draws of 64 trees over 45807 that follow 111 -> 101).  Computed once more instead.
    if constexpr (TNT > 512) asm volatile("" : "+v"(tid), "+s"(lrow));
    const int lane = tid & (WAVE - 1);
    const int wave = tid >> 6;
    const int V = a.V;
    const int k = a.k;
    const int nvec = (V + EPV - 1) / EPV;                    // the last one padded with -inf (in LDS as well)
    if (!(fabsf(ref_t) <= UNITS_MAX_REF && fabsf(ref_g) <= UNITS_MAX_REF)) return false;   // uniform
    const OnePassLayout lay = one_pass_layout(NSEG);
    ExactShared& sh = *reinterpret_cast<ExactShared*>(ex);
    double* seg = reinterpret_cast<double*>(ex + lay.seg);
    double* keep = reinterpret_cast<double*>(ex + lay.keep);
    const unsigned char* tab = tab_lds;
    AmbEntry* amb = reinterpret_cast<AmbEntry*>(ex + lay.amb);
    int* amb_count = reinterpret_cast<int*>(ex + lay.amb_count);
    UnitRow rt = unit_row(ref_t, 700.f), rg = unit_row(ref_g, 650.f);
    const float u_res32 = a.uniforms[2 * (int64_t)row + 1];  // in flight during the pass
    // the drafter's row, every load issued now; it arrives while the table and the marks are set up
    const LT* grow = reinterpret_cast<const LT*>(a.draft) + (int64_t)lrow * a.stride;
    auto draft_vector = [&](int vi) {
        if (FULL) return reinterpret_cast<const uint4*>(grow)[vi];
        if (ROWS == ROWS_WHOLE)
            return vi < nvec ? reinterpret_cast<const uint4*>(grow)[vi]
                             : make_uint4(L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD);
        return row_vector_finish<LT, EPV>(load16_any(row_vector_address<LT, EPV>(grow, vi, V)), vi, V, L::NEG_INF_WORD);
    };
    auto target_vector = [&](int vi) {
        return FULL || vi < nvec ? reinterpret_cast<const uint4*>(s_row)[vi]
                                 : make_uint4(L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD);
    };
    uint4 G[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int vi = c * TNT + tid;
        G[c] = ROWS != ROWS_ANY ? draft_vector(vi) : load16_any(row_vector_address<LT, EPV>(grow, vi, V));
    }
    if (ROWS == ROWS_ANY) {
#pragma unroll
        for (int c = 0; c < NV; ++c)
            if ((c + 1) * TNT * EPV > V) G[c] = row_vector_finish<LT, EPV>(G[c], c * TNT + tid, V, L::NEG_INF_WORD);   // uniform
    }

    // ---- table of the exponential (cache-resident), empty list ----
    for (int j = tid; j < EXP_FINE_N; j += TNT)
        reinterpret_cast<ulonglong2*>(tab_lds)[j] = make_ulonglong2(EXP_FINE[2 * j], EXP_FINE[2 * j + 1]);
    if (tid == 0) *amb_count = 0;
    __syncthreads();

    // ---- the mass of A (unnormalised); then A's tokens and xt are marked -inf in the row in LDS: t_A is zero on A
    // without the token and the token's own residual is zero in a rejected row (u g >= mass with u < 1) ----
    const int32_t* nrow = a.knn + (int64_t)xt * k;
    auto each_member = [&](auto body) {                      // entries in range: the fp32 pass has checked all k
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (tid * 4 + q < a_size && nb[q] != xt) body(nb[q]);
        for (int j = TNT * 4 + tid; j < a_size; j += TNT) {
            const int n = nrow[j];
            if (n != xt) body(n);
        }
    };
    double s_loc = 0.0;
    each_member([&](int n) { s_loc += rt.term_any(L::lds(s_row, n), tab); });
    s_loc = wave_sum(s_loc);
    if (lane == 0) sh.red[wave] = s_loc;
    // ln(Z_t / Z_g) from the fp32 sums (both finite and at least one).  Their terms are
    // 2^(l * LOG2E_F - c) with c = ref * LOG2E_F rounded to fp32, against e^(l - ref): per
    // term the two differ by (l - ref) (LOG2E_F - log2 e), which the term's error bound holds, and by
    // the rounding of c, common to the row and known exactly (the product of two floats is exact in
    // fp64): that one is put back.  Quotient and logarithm in fp64, by the last wavefront alone.
    if (tid == TNT - WAVE) {                                 // kept in LDS: registers are short during the pass
        const double LN2_D = 0.69314718055994530942;
        const double rt64 = (double)ref_t, rg64 = (double)ref_g;
        const double adj_t = ((double)(ref_t * LOG2E_F) - rt64 * (double)LOG2E_F) * LN2_D;
        const double adj_g = ((double)(ref_g * LOG2E_F) - rg64 * (double)LOG2E_F) * LN2_D;
        const double sign = log((double)Zt32 / (double)Zg32) + adj_t - adj_g + (rt64 - rg64);
        keep[0] = sign + TAU_SIGN;
        keep[1] = sign - TAU_SIGN;
    }
    if (tid == 0) {
        keep[2] = rt.start;
        keep[3] = rg.start;
        sh.bcast[0] = rt.term_any(L::lds(s_row, xt), tab);
        sh.bcast[1] = rg.term_any(lg_tok, tab);
    }
    __syncthreads();                                         // every read of a member's logit is done
    each_member([&](int n) { L::lds_set_neg_inf(s_row, n); });
    if (tid == 0) {
        double S = sh.bcast[0];
#pragma unroll
        for (int w = 0; w < TNW; ++w) S += sh.red[w];
        sh.bcast[0] = S;                                     // mass of A and the token
        L::lds_set_neg_inf(s_row, xt);
    }
    __syncthreads();

    // ---- the pass: normalisers, and per segment the terms of the certainly positive residuals ----
    OnePassAcc acc;
    acc.zt = 0.0;
    acc.zg = 0.0;
    // A rolled loop with the vectors shifted down behind it and each chunk's two sums put at the end (after the
    // last turn they are in the chunks' order): registers are indexed statically and the code stays small.
    uint32_t open = 0;                                       // bit c: a token of chunk c is not settled
    {
        const double sign_hi = keep[0], sign_lo = keep[1];
        // at most 32 tokens a turn, 16 where rows may start and end anywhere (their kernels have fewer registers left)
        constexpr int STEP = NV * EPV <= (ROWS == ROWS_ANY ? 16 : 32) ? NV : 16 / EPV;
#pragma unroll 1
        for (int c = 0; c < NV; c += STEP) {
            uint4 sums[STEP];
#pragma unroll
            for (int u = 0; u < STEP; ++u) {
                double pt, pg;
                const bool o = one_pass_vector<LT>(target_vector((c + u) * TNT + tid), G[u], rt, rg, sign_hi, sign_lo, tab,
                                                   acc, &pt, &pg);
                open |= o ? 1u << (c + u) : 0u;
                sums[u] = __builtin_bit_cast(uint4, double2{pt, pg});
            }
#pragma unroll
            for (int i = 0; i + STEP < NV; ++i) G[i] = G[i + STEP];
#pragma unroll
            for (int u = 0; u < STEP; ++u) G[NV - STEP + u] = sums[u];
        }
    }
    rt.start = keep[2];
    rg.start = keep[3];
    while (__any(open != 0)) {                               // once or so a row: which tokens, and their terms once more
        if (open) {
            const int c = __ffs((int)open) - 1;
            open &= open - 1;
#pragma unroll 1
            for (int e = 0; e < EPV; ++e) {
                const int x = (c * TNT + tid) * EPV + e;     // a token beyond V is not open, its vector may be
                const float lt = x < V ? L::lds(s_row, x) : neg_inf_f(), lg = L::glob(grow, x < V ? x : V - 1);
                const double dd = rt.arg(lt) - rg.arg(lg);
                if (dd > keep[1] && !(dd > keep[0])) {
                    const int slot = atomicAdd(amb_count, 1);
                    if (slot < AMB_CAP) {
                        amb[slot].et = rt.term(lt, tab);
                        amb[slot].eg = rg.term(lg, tab);
                        amb[slot].x = x;
                    }
                }
            }
        }
    }
    {
        double sums[2 * NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const double2 p = __builtin_bit_cast(double2, G[c]);
            sums[2 * c] = p.x;
            sums[2 * c + 1] = p.y;
        }
        wave_pair_sums<NV>(sums, lane, [&](int c, int which, double sum) { seg[2 * (c * TNW + wave) + which] = sum; });
    }
    acc.zt = wave_sum(acc.zt);
    acc.zg = wave_sum(acc.zg);
    if (lane == 0) {
        sh.red[wave] = acc.zt;
        sh.red2[wave] = acc.zg;
    }
    __syncthreads();                                         // publishes the sums, the segments and the list
    const double taken = sh.bcast[0];
    double zt = taken, zg = 0.0;                             // the marked tokens' terms are not in the sums
#pragma unroll
    for (int w = 0; w < TNW; ++w) {
        zt += sh.red[w];
        zg += sh.red2[w];
    }

    // ---- decision ----
    const double mass = taken / zt;
    const double g_tok = sh.bcast[1] / zg;
    const bool accepted = ((double)u_acc32 * g_tok < mass);
    if (tid == 0) {
        double ap;
        if (g_tok > 0.0) ap = fmin(1.0, mass / g_tok);
        else ap = mass > 0.0 ? 1.0 : 0.0;
        if (a.out_prob) a.out_prob[row] = (float)ap;
        if (a.out_mass) a.out_mass[row] = (float)mass;
        if (a.out_gtok) a.out_gtok[row] = (float)g_tok;
        if (a.out_asize) a.out_asize[row] = a_size;
        if (a.out_path) a.out_path[row] = 1;
        if (accepted) {
            a.out_accept[row] = 1;
            a.out_resample[row] = -1;
        }
    }
    if (accepted) return true;

    // ---- rejected: residual mass per segment (segments in token order), the one that holds the draw ----
    const int n_amb = *amb_count;
    const double inv_zt = 1.0 / zt, inv_zg = 1.0 / zg;
    if (wave == 0) {
        constexpr int NB = (NSEG + WAVE - 1) / WAVE;
        double incl[NB], mass_in[NB], Z = 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int s = b * WAVE + lane;
            double r = 0.0;
            if (s < NSEG) {
                r = seg[2 * s] * inv_zt - seg[2 * s + 1] * inv_zg;
                r = r > 0.0 ? r : 0.0;
                for (int i = 0; i < n_amb && i < AMB_CAP; ++i) {
                    const int v = amb[i].x / EPV;           // vector of the token: chunk v / TNT, thread v % TNT
                    if ((v / TNT) * TNW + ((v % TNT) >> 6) == s) {
                        const double d = amb[i].et * inv_zt - amb[i].eg * inv_zg;
                        r += d > 0.0 ? d : 0.0;
                    }
                }
            }
            mass_in[b] = r;
            incl[b] = Z + wave_scan_incl(r);
            Z = lane63_d(incl[b]);
        }
        const double cthr = (double)u_res32 * Z;
        int s = -1, last = 0;
        double before = 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const unsigned long long cross = __ballot(b * WAVE + lane < NSEG && incl[b] > cthr);
            const unsigned long long has = __ballot(mass_in[b] > 0.0);
            if (s < 0 && cross) {
                const int l = __ffsll((long long)cross) - 1;
                s = b * WAVE + l;
                if (l) before = __shfl(incl[b], l - 1, WAVE);
                else if (b) before = lane63_d(incl[b > 0 ? b - 1 : 0]);
                else before = 0.0;
            }
            if (has) last = b * WAVE + 63 - __clzll((long long)has);
        }
        if (s < 0) {   // rounding can leave no crossing: the last segment that holds mass takes the draw
            s = last;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (s / WAVE == b) {
                    const int l = s % WAVE;
                    before = l ? __shfl(incl[b], l - 1, WAVE) : (b ? lane63_d(incl[b > 0 ? b - 1 : 0]) : 0.0);
                }
            }
        }
        if (lane == 0) {
            sh.bcast[2] = before;   // the first two may still be read
            sh.bcast[3] = cthr;
            sh.bcast[4] = Z;
            sh.ibcast[0] = s;
        }
    }
    __syncthreads();
    // A list that overflowed, a residual without mass (by rounding), or a draw of exactly zero, which takes the first token
    // that has any residual, however far below the floors: the general path, which finds the row as it was (uniform over
    // the workgroup).
    if (n_amb > AMB_CAP || !(sh.bcast[4] > 0.0) || u_res32 == 0.f) {
        const LT* trow = reinterpret_cast<const LT*>(a.target) + (int64_t)lrow * a.stride;
        for (int j = tid; j < a_size; j += TNT) reinterpret_cast<LT*>(s_row)[nrow[j]] = trow[nrow[j]];
        if (tid == 0) reinterpret_cast<LT*>(s_row)[xt] = trow[xt];
        __syncthreads();
        return false;
    }
    // One residual term of the token-by-token evaluation: max(0, t_A(x) - g(x)), zero on A and at xt
    auto residual = [&](float lt, float lg) {
        const double d = rt.term(lt, tab) * inv_zt - rg.term(lg, tab) * inv_zg;
        return d > 0.0 ? d : 0.0;
    };
    const int ent = sh.ibcast[0];
    if (wave == (ent % TNW)) {
        const double P = sh.bcast[2], cthr = sh.bcast[3];
        const int vi = (ent / TNW) * TNT + tid;
        const int x0 = vi * EPV;
        const uint4 gv = draft_vector(vi);                   // this segment of the drafter's row, once more
        const uint4 tv = target_vector(vi);
        double r[EPV];
        double sum = 0.0;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            r[e] = residual(L::get(tv, e), L::get(gv, e));
            sum += r[e];
        }
        const double incl = wave_scan_incl(sum);
        double excl = __shfl_up(incl, 1, WAVE);
        if (lane == 0) excl = 0.0;
        const unsigned long long cross = __ballot(P + incl > cthr);
        const unsigned long long haspos = __ballot(sum > 0.0);
        // rounding between the segment's mass and its token-by-token evaluation can leave no
        // crossing lane: then the last lane that holds mass takes the draw
        const int owner = cross ? (__ffsll((long long)cross) - 1) : (haspos ? 63 - __clzll((long long)haspos) : 0);
        int found = -1;
        if (lane == owner) {
            double cum = P + excl;
            int lastpos = -1;
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                cum += r[e];
                if (r[e] > 0.0) lastpos = x0 + e;
                if (found < 0 && cum > cthr && r[e] > 0.0) found = x0 + e;
            }
            if (found < 0) found = lastpos;
        }
        found = __shfl(found, owner, WAVE);
        if (found < 0) {
            // no token of the segment holds mass: its mass was rounding noise of the sums (it takes a
            // draw within ~1e-16 of a segment edge).  The first token after it that holds mass is
            // the one the cumulative sum reaches next; failing that, the last one before it.
            const int seg_x0 = ((ent / TNW) * TNT + (ent % TNW) * WAVE) * EPV;   // first token of the segment
            int before = -1, after = INT_MAX;
            for (int x1 = 0; x1 < V; x1 += WAVE) {
                const int x = x1 + lane;
                const bool has = x < V && residual(L::lds(s_row, x < V ? x : 0), L::glob(grow, x < V ? x : 0)) > 0.0;
                const unsigned long long m = __ballot(has);
                const unsigned long long ahead = __ballot(has && x >= seg_x0), behind = m & ~ahead;
                if (ahead && after == INT_MAX) after = x1 + __ffsll((long long)ahead) - 1;
                if (behind) before = x1 + 63 - __clzll((long long)behind);
            }
            found = after != INT_MAX ? after : before;
        }
        if (lane == 0) {
            a.out_accept[row] = 0;
            a.out_resample[row] = found;
        }
    }
    return true;
}

// Per-row scalars and table slots, fetched together with the row.
struct RowMeta {
    int xt;        // draft token
    float u_acc;   // acceptance draw
    float lg_tok;  // draft logit of the token
    int nb[4];     // table slots 4*tid .. 4*tid+3 (unspecified where the slot is beyond k)
};

// fp32 path, one workgroup per row.
// TNT threads, NV 16-byte vectors per thread and row.
// VT: the token's table row can be read with 16-byte loads (k a multiple of four, table 16-byte
// aligned); the other case is a kernel of its own because a load that only one of two paths
// issues makes the hardware wait counters, which are placed statically, wait for every load.
//
// Exponentials are taken as 2^(l*log2e - c) with one reference c per row, common to all
// terms of that row, so its own rounding cancels in every comparison.  The reference is
// the maximum over the first vector slot of every thread (an eighth of the row at NV = 8)
// rather than the row maximum: any element of the row works, because the sum then holds
// a term equal to one (Z >= 1) and every term is at most Z; rows whose sum exceeds 2^46
// (an element more than 32 above the reference) are left to the exact path.
//
// first_child: in the walk that tests a node's later children against residuals only the first child of every node has
// use for a decision on the row itself; the other workgroups (half of them in trees of up to 4 children) leave here.
// The sequential step, all children decided / first ones: V = 16384 fp32, trees of 60 none of which draws, 64 trees
// 74 -> 61 us; V = 16500 fp32, 512 trees 1385 -> 1085 us; one tree of 60, where all workgroups are resident at once,
// 57 -> 54 us.
template <typename LT, int TNT, int NV, int ROWS, bool VT>
__global__ __launch_bounds__(TNT, NV > 8 ? 3 : 4) void verify_fast(VerifyArgs a) {
    using L = Lane<LT>;
    constexpr bool FULL = ROWS == ROWS_FULL;
    constexpr int EPV = L::EPV;
    constexpr int TNW = TNT / WAVE;
    // The fp64 paths' table: its place is known when the kernel is compiled, so a lookup has no base to add.
    __shared__ __align__(16) unsigned char table[EXP_FINE_BYTES];
    extern __shared__ __align__(16) unsigned char s_row[];
    const int row_bytes = (a.V * (int)sizeof(LT) + 15) & ~15;
    FastShared<TNW>& sh = *reinterpret_cast<FastShared<TNW>*>(s_row + row_bytes);
    unsigned char* ex_lds = s_row + row_bytes + sizeof(FastShared<TNW>);

    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = tid >> 6;
    const int V = a.V;
    const int k = a.k;
    const int nvec = (V + EPV - 1) / EPV;
    const int row = verification_of_block(blockIdx.x, a.N, a.row_index != nullptr);
    if (a.parent && !first_child(a.parent, a.M, row)) return;   // uniform over the workgroup
    bool row_ok;
    const int lrow = logit_row(a.row_index, a.R, row, &row_ok);

    // ---- loads, in the order their results are needed to issue further loads ----
    // Vector loads return in order.  The token comes first: the address of its table row depends on
    // it, and that second, dependent load should be in flight together with the streamed rows, not
    // start after the last of them has arrived.
    RowMeta m;
    m.xt = a.tokens[row];
    m.u_acc = a.uniforms[2 * (int64_t)row];
    // stream both rows: NV 16-byte loads per thread and row, coalesced
    uint4 T[NV], G[NV];
    {
        const LT* trow = reinterpret_cast<const LT*>(a.target) + (int64_t)lrow * a.stride;
        const LT* grow = reinterpret_cast<const LT*>(a.draft) + (int64_t)lrow * a.stride;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int vi = c * TNT + tid;
            if (FULL) {
                T[c] = load_stream16(reinterpret_cast<const uint4*>(trow) + vi);
                G[c] = load_stream16(reinterpret_cast<const uint4*>(grow) + vi);
            } else if (ROWS == ROWS_WHOLE) {
                if (vi < nvec) {
                    T[c] = load_stream16(reinterpret_cast<const uint4*>(trow) + vi);
                    G[c] = load_stream16(reinterpret_cast<const uint4*>(grow) + vi);
                } else {
                    T[c] = G[c] = make_uint4(L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD, L::NEG_INF_WORD);
                }
            } else {
                T[c] = load_stream16_any(row_vector_address<LT, EPV>(trow, vi, V));
                G[c] = load_stream16_any(row_vector_address<LT, EPV>(grow, vi, V));
            }
        }
    }
    // the token's table slots 4*tid .. 4*tid+3 and its draft logit
    {
        const int xs0 = ((unsigned)m.xt < (unsigned)V) ? m.xt : 0;
        const int32_t* nrow = a.knn + (int64_t)xs0 * k;
        const int j0 = tid * 4;
        if (VT) {        // k a multiple of four, so a thread's four slots are all inside k or all beyond
            // loaded unconditionally from a clamped slot (no branch around the load, so nothing waits
            // for it here); what threads beyond k read is never looked at (every use checks the slot
            // number against k)
            const int4 q = *reinterpret_cast<const int4*>(nrow + min(j0, k - 4));
            m.nb[0] = q.x; m.nb[1] = q.y; m.nb[2] = q.z; m.nb[3] = q.w;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) m.nb[q] = nrow[min(j0 + q, k - 1)];
        }
        m.lg_tok = L::glob(reinterpret_cast<const LT*>(a.draft) + (int64_t)lrow * a.stride, xs0);
    }
    // every load of the row is issued before anything waits for one of them
    __builtin_amdgcn_sched_barrier(0);

    {
        const int xt = m.xt;
        const bool tok_ok = (unsigned)xt < (unsigned)V;
        const int xs = tok_ok ? xt : 0;

        // ---- raw target row to LDS; reference = maximum over vector slot 0 of every thread ----
        // In the order in which the vectors arrive (left to the scheduler the first write may wait for the last load).
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int vi = c * TNT + tid;
            if (ROWS == ROWS_ANY && (c + 1) * TNT * EPV > V) {   // uniform: the chunk reaches beyond the row
                T[c] = row_vector_finish<LT, EPV>(T[c], vi, V, L::NEG_INF_WORD);
                G[c] = row_vector_finish<LT, EPV>(G[c], vi, V, L::NEG_INF_WORD);
            }
            if (FULL || vi < nvec) reinterpret_cast<uint4*>(s_row)[vi] = T[c];
            __builtin_amdgcn_sched_barrier(0);
        }
        float rt = neg_inf_f(), rg = neg_inf_f();
#pragma unroll
        for (int e = 0; e < EPV; e += 2) {
            rt = fmaxf(rt, fmaxf(L::get(T[0], e), L::get(T[0], e + 1)));
            rg = fmaxf(rg, fmaxf(L::get(G[0], e), L::get(G[0], e + 1)));
        }
        rt = wave_max(rt);
        rg = wave_max(rg);
        if (lane == 0) { sh.wmax_t[wave] = rt; sh.wmax_g[wave] = rg; }
        __syncthreads();  // the row is in LDS and the wave maxima are published
        rt = sh.wmax_t[0];
        rg = sh.wmax_g[0];
#pragma unroll
        for (int w = 1; w < TNW; ++w) {
            rt = fmaxf(rt, sh.wmax_t[w]);
            rg = fmaxf(rg, sh.wmax_g[w]);
        }
        // a sampled part without a finite logit: reference 0 (large rows then overflow and fall through)
        if (rt == neg_inf_f()) rt = 0.f;
        if (rg == neg_inf_f()) rg = 0.f;
        const float ct = rt * LOG2E_F;   // rounded once; common to every term of the row
        const float cg = rg * LOG2E_F;

        // ---- exponentials 2^(l*log2e - c), summed ----
        float st = 0.f, sg = 0.f;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            if (FULL || c * TNT < nvec) {                    // uniform; else nothing of the row in this chunk
                float et[EPV], eg[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    et[e] = hw_exp2(__builtin_fmaf(L::get(T[c], e), LOG2E_F, -ct));
                    eg[e] = hw_exp2(__builtin_fmaf(L::get(G[c], e), LOG2E_F, -cg));
                }
#pragma unroll
                for (int s = EPV / 2; s > 0; s >>= 1)
#pragma unroll
                    for (int e = 0; e < s; ++e) {
                        et[e] += et[e + s];
                        eg[e] += eg[e + s];
                    }
                st += et[0];
                sg += eg[0];
            }
        }
        st = wave_sum(st);
        sg = wave_sum(sg);

        // ---- neighbour terms of slots 4*tid .. 4*tid+3, scanned within the wavefront ----
        const SlotTerms slots = slot_terms<LT, TNT>(m.nb, xt, k, V, a.knn + (int64_t)xs * k, s_row, ct, sh.wtot, sh.wbad);
        if (lane == 0) { sh.wsum_t[wave] = st; sh.wsum_g[wave] = sg; }
        __syncthreads();  // sums and wavefront totals of the neighbour terms are published

        // ---- every wavefront: the bound on its own slots ----
        float Zt = 0.f, Zg = 0.f, woff = 0.f, run_off = 0.f;
        int bad = (tok_ok && row_ok) ? 0 : 1;
#pragma unroll
        for (int w = 0; w < TNW; ++w) {
            Zt += sh.wsum_t[w];
            Zg += sh.wsum_g[w];
            if (w < wave) woff += sh.wtot[w];
            run_off += sh.wtot[w];
            bad |= sh.wbad[w];
        }
        const float e_tx = hw_exp2(__builtin_fmaf(L::lds(s_row, xs), LOG2E_F, -ct));
        SlotTest test;
        {
            const float R = a.delta * Zt;             // divergence of the prefix, times Zt, < delta * Zt
            test.divergence = a.divergence;
            test.e_tx = e_tx;
            test.lo = R * (1.f - TAU_CUT) - ABS_SLACK;
            test.hi = R * (1.f + TAU_CUT) + ABS_SLACK;
        }
        classify_slots(slots, test, woff, WaveCut{sh.cut_np, sh.cut_df, sh.cut_s});
        __syncthreads();  // the wavefronts' results are published

        // ---- every thread: the cut, the mass, the acceptance test (same inputs, same result) ----
        int first_np = INT_MAX, first_df = INT_MAX;
        float s_cut = 0.f;
#pragma unroll
        for (int w = TNW - 1; w >= 0; --w) {
            if (sh.cut_np[w] != INT_MAX) { first_np = sh.cut_np[w]; s_cut = sh.cut_s[w]; }
            first_df = min(first_df, sh.cut_df[w]);
        }
        bool cut_definite = (first_np == INT_MAX) || (first_np == first_df);
        int a_size = (first_np == INT_MAX) ? k : first_np;
        float S = (first_np == INT_MAX) ? run_off : s_cut;
        if (first_np == INT_MAX && k > TNT * 4) {     // uniform: the walk goes on beyond four slots per thread
            if (wave == 0) {
                const CutResult tail = walk_tail<LT, TNT>(test, run_off, xt, xs, k, V, a.knn, s_row, ct);
                if (lane == 0) {
                    sh.tail[0] = tail.a_size;
                    sh.tail[1] = __float_as_int(tail.S);
                    sh.tail[2] = tail.definite ? 1 : 0;
                    sh.tail[3] = tail.bad;
                }
            }
            __syncthreads();
            a_size = sh.tail[0];
            S = __int_as_float(sh.tail[1]);
            cut_definite = sh.tail[2] != 0;
            bad |= sh.tail[3];
        }
        const float e_gx = hw_exp2(__builtin_fmaf(m.lg_tok, LOG2E_F, -cg));
        const float MA = e_tx + S;                // mass * Zt
        const float lhs = m.u_acc * e_gx * Zt;    // u * g(xt) * Zt * Zg
        const float rhs = MA * Zg;                // mass  * Zt * Zg
        const float slack = acc_slack(k);
        const bool accept = (lhs + slack) < rhs * (1.f - TAU_ACC);
        // a definite rejection settles the row only when no resampled token is asked for
        const bool reject = (a.mode == VERIFY_DECIDE) && (lhs * (1.f - TAU_ACC) > rhs + slack);
        // sums in [1, 2^46]: every term is within 32 of the reference (NaN fails both tests)
        const bool sums_ok = (Zt >= 1.f) && (Zt <= Z_MAX) && (Zg >= 1.f) && (Zg <= Z_MAX);
        const bool settled = !bad && sums_ok && cut_definite && (accept || reject);
        if (__builtin_expect(settled, 1)) {
            if (tid == 0) {
                a.out_accept[row] = accept ? 1 : 0;
                if (a.mode == VERIFY_FULL) a.out_resample[row] = -1;
                const float mass = MA / Zt;
                const float gx = e_gx / Zg;
                if (a.out_prob) a.out_prob[row] = fminf(1.f, mass / gx);
                if (a.out_mass) a.out_mass[row] = mass;
                if (a.out_gtok) a.out_gtok[row] = gx;
                if (a.out_asize) a.out_asize[row] = a_size;
                if (a.out_path) a.out_path[row] = 0;
            }
        } else {
            // not settled in fp32: this workgroup evaluates the row in fp64; the raw target row stays in
            // LDS.  With the resampled token wanted, a usable row with a definite cut is finished in one
            // pass from the registers.
            bool done = false;
            if (!bad && sums_ok && cut_definite && a.mode == VERIFY_FULL)
                done = exact_one_pass<LT, TNT, NV, ROWS>(a, row, lrow, m.nb, rt, rg, Zt, Zg, a_size, xt, m.lg_tok,
                                                         m.u_acc, table, ex_lds, s_row);
            // one call, so that it is inlined: as a function its argument block goes through memory
            if (!done) exact_row<LT, ROWS == ROWS_ANY ? ROW_ANY : ROW_WHOLE, TNT>(a, row, ex_lds, s_row, false, 0.f, 0.f, nullptr, table);
        }
    }
}

// ---------------------------------------------------------------------------
// fp64 evaluation of rows the fp32 path did not settle
// ---------------------------------------------------------------------------

// LDS the exact path needs beyond whatever precedes it: reductions, a bitmask
// of A over the vocabulary, one fp64 partial sum per (vector chunk, wavefront).
__host__ __device__ inline size_t exact_table_offset(int V, int threads = NT) {
    const size_t nvec = ((size_t)V + EXV - 1) / EXV;
    const size_t nchunk = (nvec + threads - 1) / threads;
    const size_t off = ((sizeof(ExactShared) + 15) & ~size_t(15)) + (((size_t)V + 31) / 32) * 4 + 8 +
                       nchunk * (threads / WAVE) * sizeof(double);
    return (off + 15) & ~size_t(15);
}
// ... and, last, the table of the exponential.
__host__ __device__ inline size_t exact_lds_bytes(int V, int threads = NT) {
    return exact_table_offset(V, threads) + EXP_TABLE_BYTES;
}

// One residual term: max(0, t_A(x) - g(x)) (or t_A(x) when the residual has no mass).
__device__ __forceinline__ double resid_term(int x, int xt, int V, float lt, float lg, const uint32_t* mask,
                                             double mt, double mg, double inv_zt, double inv_zg,
                                             double mass, int zero_resid, const double* tab) {
    // branch-free: both exponentials are always evaluated, then selected
    const int xm = x < V ? x : V - 1;
    const bool in_a = (x < V) && ((mask[xm >> 5] >> (xm & 31)) & 1u);
    double ta = exp_tab((double)lt - mt, tab) * inv_zt;
    ta = in_a ? 0.0 : ta;
    ta = (x == xt) ? mass : ta;
    const double gv = exp_tab((double)lg - mg, tab) * inv_zg;
    const double r = zero_resid ? ta : ta - gv;
    return r > 0.0 ? r : 0.0;
}

// Evaluates one row in fp64 with the whole workgroup.  ex: LDS region of
// exact_lds_bytes().  lds_row, lds_grow: the raw target / draft row in LDS, or null.  have_max:
// the caller has the row maxima and knows both rows are free of NaN and +inf.  tab_lds: where the exponential's table
// goes, or null: at the end of the region (exact_table_offset() bytes are enough otherwise).
// TNT: threads of the calling workgroup.  Token order of the vector layout: vector vi = chunk*TNT + tid, so (chunk,
// wavefront, lane, element) is ascending token order.  Every pass over the row
// loads the next chunk's vectors before it works on the current one.
template <typename LT, int FORM, int TNT>
__device__ __forceinline__ void exact_row(const VerifyArgs& a, int row, unsigned char* ex, const unsigned char* lds_row,
                          bool have_max, float max_t, float max_g, const unsigned char* lds_grow,
                          unsigned char* tab_lds) {
    constexpr int TNW = TNT / WAVE;
    const bool selected = a.mode == VERIFY_SELECTED;
    const int out = selected ? (int)blockIdx.x : row;   // slot of the outputs this workgroup writes
    using L = Lane<LT>;
    constexpr int EPV = EXV;
    ExactShared& sh = *reinterpret_cast<ExactShared*>(ex);
    uint32_t* mask = reinterpret_cast<uint32_t*>(ex + ((sizeof(ExactShared) + 15) & ~size_t(15)));

    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = tid >> 6;
    const int V = a.V;
    const int k = a.k;
    const int nwords = (V + 31) >> 5;
    double* tab = reinterpret_cast<double*>(tab_lds ? tab_lds : ex + exact_table_offset(V, TNT));
    for (int i = tid; i < 2 * EXP_TABLE_N; i += TNT) tab[i] = EXP_TABLE_HILO[i];   // published by the first barrier below
    double* wtot = reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(mask) + (((size_t)nwords * 4 + 7) & ~size_t(7)));
    const int nvec = (V + EPV - 1) / EPV;
    const int nchunk = (nvec + TNT - 1) / TNT;
    bool row_ok;
    const int lrow = logit_row(a.row_index, a.R, row, &row_ok);
    const LT* trow = reinterpret_cast<const LT*>(a.target) + (int64_t)lrow * a.stride;
    const LT* grow = reinterpret_cast<const LT*>(a.draft) + (int64_t)lrow * a.stride;
    const int xt = a.tokens[row];
    const double delta = (double)a.delta;
    const double u_acc = (double)a.uniforms[2 * (int64_t)row];
    const double u_res = (double)a.uniforms[2 * (int64_t)row + 1];

    // ---- usability and maxima: token and table entries in range, no NaN / +inf ----
    int bad = ((unsigned)xt < (unsigned)V) ? 0 : 1;
    const int32_t* nrow = a.knn + (int64_t)(bad ? 0 : xt) * k;
    if (!row_ok) bad = 1;
    if (!bad)
        for (int j = tid; j < k; j += TNT)
            if ((unsigned)nrow[j] >= (unsigned)V) bad = 1;
    float mtf = neg_inf_f(), mgf = neg_inf_f();
    if (have_max) {
        mtf = max_t;
        mgf = max_g;
    } else {
        float tn[EPV], gn[EPV];
        VecLoad<LT, FORM>::load(trow, lds_row, tid, V, tn);
        VecLoad<LT, FORM>::load(grow, lds_grow, tid, V, gn);
        for (int c = 0; c < nchunk; ++c) {
            float tf[EPV], gf[EPV];
#pragma unroll
            for (int e = 0; e < EPV; ++e) { tf[e] = tn[e]; gf[e] = gn[e]; }
            if (c + 1 < nchunk) {
                VecLoad<LT, FORM>::load(trow, lds_row, (c + 1) * TNT + tid, V, tn);
                VecLoad<LT, FORM>::load(grow, lds_grow, (c + 1) * TNT + tid, V, gn);
            }
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                if (isnan(tf[e]) || isnan(gf[e]) || tf[e] == INFINITY || gf[e] == INFINITY) bad = 1;
                mtf = fmaxf(mtf, tf[e]);
                mgf = fmaxf(mgf, gf[e]);
            }
        }
    }
    const double mt = block_max<TNW>((double)mtf, sh.red, tid);
    const double mg = block_max<TNW>((double)mgf, sh.red2, tid);
    if (mt == -INFINITY || mg == -INFINITY) bad = 1;
    bad = block_or_i<TNW>(bad, sh.ired, tid);
    if (bad) {
        if (tid == 0) {
            if (selected) {
                a.out_resample[out] = -2;
            } else {
                a.out_accept[row] = -1;
                if (a.mode == VERIFY_FULL) a.out_resample[row] = -1;
                if (a.out_prob) a.out_prob[row] = NAN;
                if (a.out_mass) a.out_mass[row] = NAN;
                if (a.out_gtok) a.out_gtok[row] = NAN;
                if (a.out_asize) a.out_asize[row] = -1;
                if (a.out_path) a.out_path[row] = 1;
            }
        }
        return;
    }

    // ---- softmax normalisers ----
    double zt = 0.0, zg = 0.0;
    {
        float tn[EPV], gn[EPV];
        VecLoad<LT, FORM>::load(trow, lds_row, tid, V, tn);
        VecLoad<LT, FORM>::load(grow, lds_grow, tid, V, gn);
        for (int c = 0; c < nchunk; ++c) {
            float tf[EPV], gf[EPV];
#pragma unroll
            for (int e = 0; e < EPV; ++e) { tf[e] = tn[e]; gf[e] = gn[e]; }
            if (c + 1 < nchunk) {
                VecLoad<LT, FORM>::load(trow, lds_row, (c + 1) * TNT + tid, V, tn);
                VecLoad<LT, FORM>::load(grow, lds_grow, (c + 1) * TNT + tid, V, gn);
            }
            double st = 0.0, sg = 0.0;
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                st += exp_tab((double)tf[e] - mt, tab);
                sg += exp_tab((double)gf[e] - mg, tab);
            }
            zt += st;
            zg += sg;
        }
    }
    zt = block_sum<TNW>(zt, sh.red, tid);
    zg = block_sum<TNW>(zg, sh.red2, tid);

    // ---- nearest-first walk over the table row ----
    const double t_tok = exp_tab((double)L::glob(trow, xt) - mt, tab) / zt;
    int a_size;
    double S;
    exact_walk<LT, TNT>(trow, lds_row, nrow, k, xt, mt, zt, a.divergence, t_tok, delta, sh, tid, &a_size, &S, tab);

    const double g_tok = exp_tab((double)L::glob(grow, xt) - mg, tab) / zg;
    const double mass = t_tok + S;
    const bool accepted = (u_acc * g_tok < mass);
    if (tid == 0 && !selected) {
        double ap;
        if (g_tok > 0.0) ap = fmin(1.0, mass / g_tok);
        else ap = mass > 0.0 ? 1.0 : 0.0;
        if (a.out_prob) a.out_prob[row] = (float)ap;
        if (a.out_mass) a.out_mass[row] = (float)mass;
        if (a.out_gtok) a.out_gtok[row] = (float)g_tok;
        if (a.out_asize) a.out_asize[row] = a_size;
        if (a.out_path) a.out_path[row] = 1;
    }
    if (accepted || a.mode == VERIFY_DECIDE) {
        if (tid == 0) {
            if (selected) {
                a.out_resample[out] = -1;
            } else {
                a.out_accept[row] = accepted ? 1 : 0;
                if (a.mode == VERIFY_FULL) a.out_resample[row] = -1;
            }
        }
        return;
    }

    // ---- rejected: distorted target t_A, residual max(0, t_A - g), inverse CDF ----
    for (int w = tid; w < nwords; w += TNT) mask[w] = 0u;
    __syncthreads();
    for (int j = tid; j < a_size; j += TNT) {
        const int n = nrow[j];
        if (n != xt) atomicOr(&mask[n >> 5], 1u << (n & 31));
    }
    __syncthreads();

    const double inv_zt = 1.0 / zt, inv_zg = 1.0 / zg;
    int zero_resid = 0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        // per (chunk, wavefront) partial sums of the residual, in token order
        {
            float tn[EPV], gn[EPV];
            VecLoad<LT, FORM>::load(trow, lds_row, tid, V, tn);
            VecLoad<LT, FORM>::load(grow, lds_grow, tid, V, gn);
            for (int c = 0; c < nchunk; ++c) {
                const int vi = c * TNT + tid;
                float tf[EPV], gf[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) { tf[e] = tn[e]; gf[e] = gn[e]; }
                if (c + 1 < nchunk) {
                    VecLoad<LT, FORM>::load(trow, lds_row, vi + TNT, V, tn);
                    VecLoad<LT, FORM>::load(grow, lds_grow, vi + TNT, V, gn);
                }
                double s = 0.0;
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    s += resid_term(vi * EPV + e, xt, V, tf[e], gf[e], mask, mt, mg, inv_zt, inv_zg, mass,
                                    zero_resid, tab);
                s = wave_sum(s);
                if (lane == 0) wtot[c * TNW + wave] = s;
            }
        }
        __syncthreads();
        // every wavefront scans the partial sums itself, 64 entries at a time in token order
        const int nent = nchunk * TNW;
        double Z = 0.0;
        for (int base = 0; base < nent; base += WAVE) Z += wave_sum(base + lane < nent ? wtot[base + lane] : 0.0);
        if (!(Z > 0.0) && !zero_resid) {  // residual without mass: sample t_A itself
            zero_resid = 1;
            __syncthreads();
            continue;
        }
        const double cthr = u_res * Z;
        // first (chunk, wavefront) whose running sum exceeds the threshold; P: the sum before it
        double P = 0.0;
        int ent = -1;
        for (int base = 0; base < nent && ent < 0; base += WAVE) {
            const double incl = P + wave_scan_incl(base + lane < nent ? wtot[base + lane] : 0.0);
            const unsigned long long cross = __ballot(base + lane < nent && incl > cthr);
            if (cross) {
                const int l = __ffsll((long long)cross) - 1;
                ent = base + l;
                P = l ? __shfl(incl, l - 1, WAVE) : P;
            } else {
                P = __shfl(incl, WAVE - 1, WAVE);
            }
        }
        if (ent < 0) {   // rounding left no crossing: the last entry takes the draw
            ent = nent - 1;
            P -= wtot[ent];
        }
        if (wave == (ent % TNW)) {
            const int c = ent / TNW;
            const int vi = c * TNT + tid;
            float tf[EPV], gf[EPV];
            VecLoad<LT, FORM>::load(trow, lds_row, vi, V, tf);
            VecLoad<LT, FORM>::load(grow, lds_grow, vi, V, gf);
            double r[EPV];
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                r[e] = resid_term(vi * EPV + e, xt, V, tf[e], gf[e], mask, mt, mg, inv_zt, inv_zg, mass, zero_resid, tab);
                s += r[e];
            }
            const double incl = wave_scan_incl(s);
            double excl = __shfl_up(incl, 1, WAVE);
            if (lane == 0) excl = 0.0;
            const unsigned long long cross = __ballot(P + incl > cthr);
            const unsigned long long haspos = __ballot(s > 0.0);
            // rounding between the butterfly sum and the scan can leave no crossing lane:
            // then the last lane that holds mass takes the draw
            const int owner = cross ? (__ffsll((long long)cross) - 1)
                                    : (haspos ? 63 - __clzll((long long)haspos) : 0);
            if (lane == owner) {
                double cum = P + excl;
                int found = -1, lastpos = -1;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    cum += r[e];
                    if (r[e] > 0.0) lastpos = vi * EPV + e;
                    if (found < 0 && cum > cthr && r[e] > 0.0) found = vi * EPV + e;
                }
                if (found < 0) found = lastpos;
                if (!selected) a.out_accept[row] = 0;
                a.out_resample[out] = found;
            }
        }
        break;
    }
}

// Every row through the exact path: for shapes the fast path does not cover.
template <typename LT>
__global__ __launch_bounds__(NT) void verify_exact(VerifyArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int row = verification_of_block(blockIdx.x, a.N, a.row_index != nullptr);
    if (a.parent && !first_child(a.parent, a.M, row)) return;
    exact_row<LT, ROW_ELEMENTS>(a, row, smem, nullptr, false, 0.f, 0.f);
}

// VERIFY_SELECTED: workgroup i evaluates verification select[i] and writes out_resample[i].
// Few rows per launch, so each gets a workgroup of 512 threads (two wavefronts per SIMD, no register
// spills; 1024 threads measured slower): the fp64 passes of a row are
// latency-bound at one wavefront per SIMD.
constexpr int SEL_NT = 512;
// Evaluates verification v in fp64 with all threads of this workgroup (VERIFY_SELECTED: only
// out_resample[blockIdx.x] is written).  When they fit, both logit rows are first copied into LDS,
// all loads in flight together, so the fp64 passes read LDS.
template <typename LT, bool VEC>
__device__ __forceinline__ void selected_row(const VerifyArgs& a, int v, unsigned char* smem) {
    const unsigned char* lds_t = nullptr;
    const unsigned char* lds_g = nullptr;
    if (VEC && a.stage_rows) {
        const int row_bytes = a.V * (int)sizeof(LT);          // a multiple of 8 (VEC: V % 4 == 0)
        const size_t ex_bytes = (exact_lds_bytes(a.V, SEL_NT) + 15) & ~size_t(15);
        unsigned char* st = smem + ex_bytes;
        unsigned char* sg = st + ((row_bytes + 15) & ~15);
        bool row_ok;
        const int lrow = logit_row(a.row_index, a.R, v, &row_ok);
        const uint2* tsrc = reinterpret_cast<const uint2*>(reinterpret_cast<const LT*>(a.target) + (int64_t)lrow * a.stride);
        const uint2* gsrc = reinterpret_cast<const uint2*>(reinterpret_cast<const LT*>(a.draft) + (int64_t)lrow * a.stride);
        const int n8 = row_bytes >> 3;
        for (int i = threadIdx.x; i < n8; i += SEL_NT) {
            reinterpret_cast<uint2*>(st)[i] = tsrc[i];
            reinterpret_cast<uint2*>(sg)[i] = gsrc[i];
        }
        __syncthreads();
        lds_t = st;
        lds_g = sg;
    }
    exact_row<LT, VEC ? ROW_WHOLE : ROW_ELEMENTS, SEL_NT>(a, v, smem, lds_t, false, 0.f, 0.f, lds_g);
}

// VERIFY_SELECTED: workgroup i evaluates verification select[i] and writes out_resample[i].
template <typename LT, bool VEC>
__global__ __launch_bounds__(SEL_NT) void resample_selected(VerifyArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int v = a.select[blockIdx.x];
    if (v < 0 || v >= a.N) {   // uniform per workgroup
        if (threadIdx.x == 0) a.out_resample[blockIdx.x] = v < 0 ? v : -2;
        return;
    }
    selected_row<LT, VEC>(a, v, smem);
}

// Second half of a tree step: workgroup b walks tree b over the decisions in a.out_accept (its
// first wavefront), then draws the one residual the walk asks for and writes a.out_resample[b].
template <typename LT, bool VEC>
__global__ __launch_bounds__(SEL_NT) void tree_finish(VerifyArgs a, const int32_t* parent, int M, int32_t* out_len,
                                                      int32_t* out_path) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tree = blockIdx.x;
    int32_t* path = out_path + (int64_t)tree * M;
    int* bcast = reinterpret_cast<int*>(smem);
    if (threadIdx.x < WAVE) {
        int len;
        const int next = walk_tree(a.out_accept + (int64_t)tree * M, nullptr, parent + (int64_t)tree * M, M, tree,
                                   path, &len);
        for (int j = len + threadIdx.x; j < M; j += WAVE) path[j] = -1;
        if (threadIdx.x == 0) {
            out_len[tree] = len;
            bcast[0] = next;
        }
    }
    __syncthreads();
    const int v = bcast[0];
    __syncthreads();              // the exact path reuses this LDS
    if (v < 0) {                  // uniform per workgroup: nothing to resample
        if (threadIdx.x == 0) a.out_resample[tree] = v;
        return;
    }
    selected_row<LT, VEC>(a, v, smem);
}

// ---------------------------------------------------------------------------
// host-side launch
// ---------------------------------------------------------------------------

// Dynamic LDS of verify_fast: raw row, reductions, then the exact paths' region.  (Beside it: EXP_FINE_BYTES of the table.)
template <typename LT>
static size_t fast_lds_bytes(int V, int threads, int nv) {
    const size_t row_bytes = ((size_t)V * sizeof(LT) + 15) & ~size_t(15);
    const size_t head = threads == 256 ? sizeof(FastShared<4>) : threads == 512 ? sizeof(FastShared<8>) : sizeof(FastShared<16>);
    const size_t one_pass = one_pass_layout(nv * (threads / WAVE)).total;
    const size_t exact = exact_table_offset(V, threads);
    return row_bytes + head + (one_pass > exact ? one_pass : exact);
}

// Rows of 16-byte aligned whole vectors, stride included.
template <typename LT>
static bool whole_vectors(const VerifyArgs& a) {
    const uintptr_t align = reinterpret_cast<uintptr_t>(a.target) | reinterpret_cast<uintptr_t>(a.draft) |
                            (uintptr_t)(a.stride * (int64_t)sizeof(LT));
    return (align & 15) == 0 && a.V % Lane<LT>::EPV == 0;
}

// The table can be read with 16-byte loads: four slots of a thread at a time.
static bool vector_table(const VerifyArgs& a) {
    return (a.k & 3) == 0 && (reinterpret_cast<uintptr_t>(a.knn) & 15) == 0;
}

// launch == false: only the LDS limits are raised (lantern_prepare), nothing is enqueued.
// OTHER: what the kernels for rows that do not fill every slot know (ROWS_WHOLE or ROWS_ANY).
template <typename LT, int TNT, int NV, int OTHER = ROWS_ANY>
static hipError_t launch_fast_nv(const VerifyArgs& a, hipStream_t stream, bool launch) {
    const size_t lds = fast_lds_bytes<LT>(a.V, TNT, NV);
    const bool full = a.V == NV * TNT * Lane<LT>::EPV && whole_vectors<LT>(a);
    // three instantiations: full rows with a vector-readable table, other rows with one, and the rest
    const bool vt = vector_table(a);
    if (!launch) {   // every one of them may be needed later
        hipError_t e = allow_lds<&verify_fast<LT, TNT, NV, ROWS_FULL, true>>(lds);
        if (e == hipSuccess) e = allow_lds<&verify_fast<LT, TNT, NV, OTHER, true>>(lds);
        if (e == hipSuccess) e = allow_lds<&verify_fast<LT, TNT, NV, OTHER, false>>(lds);
        return e;
    }
    const hipError_t e = (full && vt) ? allow_lds<&verify_fast<LT, TNT, NV, ROWS_FULL, true>>(lds)
                         : vt         ? allow_lds<&verify_fast<LT, TNT, NV, OTHER, true>>(lds)
                                      : allow_lds<&verify_fast<LT, TNT, NV, OTHER, false>>(lds);
    if (e != hipSuccess) return e;
    if (full && vt)
        hipLaunchKernelGGL((verify_fast<LT, TNT, NV, ROWS_FULL, true>), dim3(a.N), dim3(TNT), lds, stream, a);
    else if (vt)
        hipLaunchKernelGGL((verify_fast<LT, TNT, NV, OTHER, true>), dim3(a.N), dim3(TNT), lds, stream, a);
    else
        hipLaunchKernelGGL((verify_fast<LT, TNT, NV, OTHER, false>), dim3(a.N), dim3(TNT), lds, stream, a);
    return hipGetLastError();
}

// Rows of 32 to 64 KiB: 256 threads with 16 vectors each instead of 512 with 8.  A row that is rejected in fp64
// is done sooner by 512 threads (its workgroup is what the launch waits for); rows that are only read in fp32 pass
// faster through 256 where that lets a compute unit hold three workgroups instead of two (three rows in LDS, three
// wavefronts per SIMD), and where every slot is filled.  Measured, 512 threads against 256:
//   decisions, 3840 rows of 9000 fp32     58.7 / 48.4 us    60 rows 8.0 / 7.6       three fit
//   decisions, 3840 rows of 32768 bf16    88.3 / 82.8       60 rows 9.6 / 9.2       full
//   decisions, 3840 rows of 24576 bf16    75.5 / 75.3       60 rows 9.0 / 9.2       neither
//   tokens too, 45 % rejected: 3840 rows of 9000 fp32 177 / 157, 60 rows 23.1 / 28.5      three fit
//                              3840 rows of 24576 bf16 245 / 285, 60 rows 32.9 / 43.1     two fit
// So decisions take 256 in the first two cases, tokens where three fit and there are more rows than two per unit.
// Only aligned whole vectors: at any other address the 16 vectors do not fit three wavefronts' registers.
constexpr int COMPUTE_UNITS = 256;
constexpr size_t LDS_OF_A_UNIT = 160 * 1024;
template <typename LT>
static bool fewer_threads(const VerifyArgs& a) {
    if (!whole_vectors<LT>(a)) return false;
    const bool three = 3 * (fast_lds_bytes<LT>(a.V, NT, 16) + EXP_FINE_BYTES) <= LDS_OF_A_UNIT;
    if (a.mode == VERIFY_DECIDE) return three || (a.V == 16 * NT * Lane<LT>::EPV && vector_table(a));
    return three && a.N > 2 * COMPUTE_UNITS;
}

// Up to 8 vectors per thread and row stay in registers; the number of threads follows from that, so a
// longer row takes a larger workgroup (V = 65536 bf16, 960 rows of which 45 % are rejected: 230 us with
// 1024 threads against 527 us on the fp64 path that such rows took before; 960 rows of 8192 bf16 logits
// at addresses not aligned to 16 bytes: 35 us against 68 us).
template <typename LT>
static hipError_t launch_fast(const VerifyArgs& a, hipStream_t stream, bool launch) {
    const int nvec = (a.V + Lane<LT>::EPV - 1) / Lane<LT>::EPV;
    const int nv = (nvec + NT - 1) / NT;
    if (nv <= 1) return launch_fast_nv<LT, 256, 1>(a, stream, launch);
    if (nv <= 2) return launch_fast_nv<LT, 256, 2>(a, stream, launch);
    if (nv <= 4) return launch_fast_nv<LT, 256, 4>(a, stream, launch);
    if (nv <= 8) return launch_fast_nv<LT, 256, 8>(a, stream, launch);
    if (nv <= 16) {
        if (launch)
            return fewer_threads<LT>(a) ? launch_fast_nv<LT, 256, 16, ROWS_WHOLE>(a, stream, true)
                                        : launch_fast_nv<LT, 512, 8>(a, stream, true);
        const hipError_t e = launch_fast_nv<LT, 256, 16, ROWS_WHOLE>(a, stream, false);
        return e == hipSuccess ? launch_fast_nv<LT, 512, 8>(a, stream, false) : e;
    }
    return launch_fast_nv<LT, 1024, 8>(a, stream, launch);
}

// Rows the fp32 pass covers: at least one 16-byte vector, at most 8 vectors for each of 1024 threads,
// k within the scan's depth.
template <typename LT>
static bool fast_shape(int V, int k) {
    constexpr int EPV = Lane<LT>::EPV;
    return V >= EPV && V <= 8 * 1024 * EPV && k <= FAST_MAX_K;
}

template <typename LT>
static hipError_t launch_typed(const VerifyArgs& a, hipStream_t stream) {
    // Diagnostics of rows that are no whole vectors, or of more than 64 KiB, come from the fp64 path as
    // they always have; decisions and tokens are the same either way.
    const bool diagnostics = a.out_prob || a.out_mass || a.out_gtok;
    const bool long_row = (a.V + Lane<LT>::EPV - 1) / Lane<LT>::EPV > 16 * NT;
    if (fast_shape<LT>(a.V, a.k) && !(diagnostics && (long_row || !whole_vectors<LT>(a))))
        return launch_fast<LT>(a, stream, true);
    const size_t lds = exact_lds_bytes(a.V);
    const hipError_t e = allow_lds<&verify_exact<LT>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((verify_exact<LT>), dim3(a.N), dim3(NT), lds, stream, a);
    return hipGetLastError();
}

// LDS of the 512-thread kernels; *stage: both logit rows fit beside the exact path's data.
template <typename LT>
static size_t selected_lds_bytes(int V, bool vec, int* stage) {
    const size_t lds = exact_lds_bytes(V, SEL_NT);
    const size_t staged = ((lds + 15) & ~size_t(15)) + 2 * (((size_t)V * sizeof(LT) + 15) & ~size_t(15));
    *stage = (vec && staged <= 150 * 1024) ? 1 : 0;
    return *stage ? staged : lds;
}

template <typename LT>
static hipError_t launch_selected_typed(const VerifyArgs& a_in, const int32_t* parent, int M, int32_t* out_len,
                                        int32_t* out_path, hipStream_t stream) {
    VerifyArgs a = a_in;
    const uintptr_t align = reinterpret_cast<uintptr_t>(a.target) | reinterpret_cast<uintptr_t>(a.draft) |
                            (uintptr_t)(a.stride * (int64_t)sizeof(LT));
    const bool vec = (align & 15) == 0 && (a.V % EXV) == 0;   // rows 16-byte aligned, whole vectors
    const size_t lds = selected_lds_bytes<LT>(a.V, vec, &a.stage_rows);
    if (parent) {   // walk and draw in one launch, one workgroup per tree
        const hipError_t e = vec ? allow_lds<&tree_finish<LT, true>>(lds) : allow_lds<&tree_finish<LT, false>>(lds);
        if (e != hipSuccess) return e;
        if (vec)
            hipLaunchKernelGGL((tree_finish<LT, true>), dim3(a.n_sel), dim3(SEL_NT), lds, stream, a, parent, M, out_len,
                               out_path);
        else
            hipLaunchKernelGGL((tree_finish<LT, false>), dim3(a.n_sel), dim3(SEL_NT), lds, stream, a, parent, M, out_len,
                               out_path);
        return hipGetLastError();
    }
    const hipError_t e = vec ? allow_lds<&resample_selected<LT, true>>(lds) : allow_lds<&resample_selected<LT, false>>(lds);
    if (e != hipSuccess) return e;
    if (vec)
        hipLaunchKernelGGL((resample_selected<LT, true>), dim3(a.n_sel), dim3(SEL_NT), lds, stream, a);
    else
        hipLaunchKernelGGL((resample_selected<LT, false>), dim3(a.n_sel), dim3(SEL_NT), lds, stream, a);
    return hipGetLastError();
}

// Raises, on the current device, the LDS limit of every kernel a verification of this vocabulary
// size and logit type can launch, whatever the alignment of the caller's buffers turns out to be.
template <typename LT>
static hipError_t prepare_typed(int V, int k) {
    // the runtime defers loading a file's kernels to their first use: make that happen now
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&verify_exact<LT>));
    if (e != hipSuccess) return e;
    if (fast_shape<LT>(V, k)) {
        VerifyArgs a{};
        a.V = V;
        a.k = k;
        e = launch_fast<LT>(a, nullptr, false);
    }
    if (e == hipSuccess) e = allow_lds<&verify_exact<LT>>(exact_lds_bytes(V));
    for (int vec = 0; vec < 2 && e == hipSuccess; ++vec) {
        if (vec && (V % EXV) != 0) break;
        int stage;
        const size_t lds = selected_lds_bytes<LT>(V, vec != 0, &stage);
        if (vec) {
            e = allow_lds<&tree_finish<LT, true>>(lds);
            if (e == hipSuccess) e = allow_lds<&resample_selected<LT, true>>(lds);
        } else {
            e = allow_lds<&tree_finish<LT, false>>(lds);
            if (e == hipSuccess) e = allow_lds<&resample_selected<LT, false>>(lds);
        }
    }
    return e;
}

hipError_t prepare_verify(int logits_dtype, int V, int k) {
    return logits_dtype == 0 ? prepare_typed<float>(V, k) : prepare_typed<uint16_t>(V, k);
}

hipError_t launch_resample_selected(const VerifyArgs& a, int logits_dtype, hipStream_t stream) {
    if (logits_dtype == 0) return launch_selected_typed<float>(a, nullptr, 0, nullptr, nullptr, stream);
    return launch_selected_typed<uint16_t>(a, nullptr, 0, nullptr, nullptr, stream);
}

// Which kernel ends a plain tree step.  The one that keeps the row pair in registers and evaluates every
// exponential once (1024 threads, the target in LDS as doubles: one workgroup to a compute unit beyond some 9000
// tokens) against tree_finish (512 threads, several passes over rows staged in LDS, or read element by element
// where they are not aligned whole vectors).  Time after the decisions, 60 candidates a tree, tree_finish / registers:
//   V     aligned bf16, 1 / 64 / 512 trees       aligned fp32, 1 / 64 / 512          not aligned, about V, fp32
//   1024  10.1 11.0 19.6 / 12.1 13.1 27.4 us     6.7 11.4 19.2 / 7.7 13.4 28.6       6.7 12.5 24.6 / 7.5 13.1 29.4
//   2048                                                                              15.0 18.1 30.7 / 12.8 13.9 33.6
//   4096  8.3 14.6 27.6 / 8.7 15.4 33.4          8.0 14.6 28.4 / 8.7 15.6 35.6       10.6 22.1 33.8 / 9.5 17.4 44.5
//   8192  10.9 20.0 35.4 / 10.7 19.8 44.2        10.6 21.5 36.2 / 10.8 20.4 42.1     22.1 31.9 36.5 / 19.4 22.3 59.5
//   9216  21.2 23.0 45.8 / 19.4 21.1 49.4        21.0 24.9 41.7 / 19.7 22.5 50.6
//  12288  25.1 30.1 39.6 / 21.4 23.5 49.2        25.3 32.3 61.0 / 21.9 24.3 52.1     32.3 41.7 52.2 / 22.1 26.2 61.1
//  16384  30.4 35.0 55.1 / 24.2 27.7 49.5        30.3 36.0 74.2 / 24.5 27.5 53.1     17.2 46.7 81.1 / 14.5 30.6 55.3
// Trees whose walk ends without a draw take 3 to 6 us in either.  So: registers beyond 8192 tokens (2048 where rows
// are not aligned) as long as every tree has a compute unit, and beyond 12288 for any number of trees.
static bool draw_from_registers(const VerifyArgs& a, size_t logit_bytes) {
    if (!tree_plain_fits(a.V)) return false;
    if (a.V > 12288) return true;
    const uintptr_t align = reinterpret_cast<uintptr_t>(a.target) | reinterpret_cast<uintptr_t>(a.draft) |
                            (uintptr_t)(a.stride * (int64_t)logit_bytes);
    const bool whole = (align & 15) == 0 && a.V % EXV == 0;
    return a.n_sel <= COMPUTE_UNITS && a.V > (whole ? 8192 : 2048);
}

hipError_t launch_tree_finish(const VerifyArgs& a, const int32_t* parent, int M, int32_t* out_len, int32_t* out_path,
                              int logits_dtype, hipStream_t stream) {
    if (draw_from_registers(a, logits_dtype == 0 ? sizeof(float) : sizeof(uint16_t))) {
        SequentialArgs s{};
        s.target = a.target;
        s.draft = a.draft;
        s.R = a.R;
        s.V = a.V;
        s.stride = a.stride;
        s.row_index = a.row_index;
        s.parent = parent;
        s.B = a.n_sel;
        s.M = M;
        s.tokens = a.tokens;
        s.knn = a.knn;
        s.k = a.k;
        s.divergence = a.divergence;
        s.delta = a.delta;
        s.uniforms = a.uniforms;
        s.accept = a.out_accept;
        s.out_len = out_len;
        s.out_path = out_path;
        s.out_next = a.out_resample;
        return launch_trees_plain(s, logits_dtype, stream);
    }
    if (logits_dtype == 0) return launch_selected_typed<float>(a, parent, M, out_len, out_path, stream);
    return launch_selected_typed<uint16_t>(a, parent, M, out_len, out_path, stream);
}

hipError_t launch_verify(const VerifyArgs& a, int logits_dtype, hipStream_t stream) {
    if (logits_dtype == 0) return launch_typed<float>(a, stream);
    return launch_typed<uint16_t>(a, stream);
}

}  // namespace lantern
