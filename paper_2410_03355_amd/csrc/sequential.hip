// Walk of draft trees under the sequential-residual sibling rule (Section 2, Algorithm 1 applied
// to the several candidates a tree offers for one position; Section 4.3 for each candidate).
//
// Standing at a node, its children are tried in index order on the logit rows of the first child:
//     t_1 = softmax(target row)
//     child j: the relaxed verification of Section 4.3 with t_j in place of the target;
//              accepted: the walk moves to that child;
//              rejected: t_{j+1} = max(0, t_{j,A} - g) / Z, the residual of that verification
//     every child rejected: the token that follows is drawn from the last residual.
// With k = 1 or delta = 0 this is recursive rejection sampling, which keeps the target law.
//
// The chain t_1, t_2, ... is sequential, so one workgroup of 1024 threads walks one tree and keeps
// the current target and the drafter's distribution in fp64 (unnormalised terms and a scale each: no
// division per token).  The test of a group's first child is the plain verification of that
// candidate, so its decision is read from the row-parallel pass (lantern_decide_rows over the first
// children, launched first): only groups whose first child is rejected build the vectors.
// A launch has as many workgroups as trees and each is a chain of passes over the vocabulary, so what
// counts is the length of that chain:
//   - a thread owns pairs of neighbouring tokens (4-byte loads of bf16, 8-byte loads of fp32, 16-byte
//     LDS accesses), the same ones in every pass, a wavefront a contiguous part of the vocabulary; the
//     drafter's terms then stay in registers and the rows are read from memory once;
//   - the current target is gathered at random by the neighbourhood walk: it lives in LDS;
//   - one pass per rejected child forms its residual and adds it up, storing what is not positive with
//     its sign turned (t_{j,A} is needed again when the residual turns out to have no mass);
//   - the residual draw is taken once per group, after its last child, by the one wavefront whose part
//     of the vocabulary holds it;
//   - a tree's parents, tokens, decisions and draws are staged in LDS, and every wavefront looks for the
//     next child by itself.
// A group's pairs of logits and, in their room, the drafter's terms take 4 registers per step; the Jensen-Shannon
// bound's logarithms are a function call, over which few registers live, in kernels of their own.  So the walk under
// total variation keeps out of scratch memory: setting that up is 1 to 3 us of every walk (64 trees none of which draws,
// V = 8192 fp32: 43.6 -> 39.7 us the step) and the spilled terms more (V = 16384 fp32, 64 trees: 163 -> 148 us).
// The exponentials (two rows of them per group, on one compute unit: 6 of a plain draw's 21 us) are those of the one-pass
// evaluation, 17 instructions each with the subtraction of the maximum, and what is the same in all lanes is kept
// in scalar registers: V = 16384 bf16, 64 trees, 90 -> 83 us the walk, 26.6 -> 23.9 the plain draw; with the table an LDS object whose
// place the compiler knows 87 -> 80 and 23.6 -> 22.2.
// Second half of the plain step (PLAIN): its first wavefront walks the tree over the decisions as every other walk
// does (tree_walk.h), then the workgroup evaluates the one candidate whose draw is wanted.  V = 16384 bf16, 1 / 64
// trees that draw: 20 / 22 us, without a draw 4 us (24 / 28 with the exponentials before); 27 / 31 and 10 us with the search for children among the passes.
// Vocabularies that do not fit in LDS keep both vectors in the workspace.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include "device_utils.h"
#include "exp64.h"
#include "exp_table.h"
#include "lds_limit.h"
#include "sequential_args.h"
#include "tree_walk.h"
#include "verify_common.h"

namespace lantern {

constexpr int SNT = 1024;
constexpr int SNW = SNT / WAVE;
constexpr int PAIR_STEP = 2 * WAVE;   // tokens of one step of a wavefront: a pair per lane
constexpr int SNODES = 128;           // nodes of a tree that are staged in LDS; larger trees are read in place

// Two neighbouring logits with one load from an address aligned to the element only, and the two words that
// hold them afterwards: the logits as fp32, later a double.
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
template <typename LT> struct RawPair;
template <> struct RawPair<float> {
    typedef uint32_t raw __attribute__((ext_vector_type(2), aligned(4)));
    __device__ static __forceinline__ u2 words(raw v) { return u2{v.x, v.y}; }
    __device__ static __forceinline__ raw twice(const float* p) {
        const uint32_t w = __float_as_uint(*p);
        return raw{w, w};
    }
};
template <> struct RawPair<uint16_t> {
    typedef uint32_t raw __attribute__((aligned(2)));
    __device__ static __forceinline__ u2 words(raw v) { return u2{v << 16, v & 0xFFFF0000u}; }
    __device__ static __forceinline__ raw twice(const uint16_t* p) { return *p * 0x10001u; }
};
__device__ __forceinline__ float lo_of(u2 v) { return __uint_as_float(v.x); }
__device__ __forceinline__ float hi_of(u2 v) { return __uint_as_float(v.y); }
__device__ __forceinline__ double double_of(u2 v) { return __hiloint2double((int)v.y, (int)v.x); }
__device__ __forceinline__ u2 words_of(double d) { return u2{(uint32_t)__double2loint(d), (uint32_t)__double2hiint(d)}; }
// An integer whose origin the compiler does not see: what is computed from it stays where it is used
// (token numbers and bounds of every step, hoisted out of the walk, would take more registers than there are).
__device__ __forceinline__ int opaque_int(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
// A function of its own: its logarithms' constants would occupy registers all through the walk.
__device__ __noinline__ bool jsd_fails(double t_tok, double moved, double delta) {
    return !(prefix_divergence64(1, t_tok, moved) < delta);
}
typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));

struct SeqShared {
    alignas(16) uint64_t tab[2 * EXP_FINE_N];
    double sum_a[SNW], sum_b[SNW];   // softmax sums, then the walk's totals and sums before its cut
    double wr[SNW], wt[SNW];         // residual mass and distorted target's mass of every wavefront's part
    float mt[SNW], mg[SNW];
    int bad[SNW], cut[SNW];
    int ired[SNW];
    int drawn;
    int parent[SNODES], row[SNODES], token[SNODES], accept[SNODES];
    float u_acc[SNODES], u_res[SNODES];
};

// NP > 0: every wavefront's part of the vocabulary is at most NP steps; the current target lives in LDS
// and the drafter's terms in registers.  NP == 0: any vocabulary, both vectors in the workspace.
// PLAIN: the second half of the plain tree step instead (NP > 0, no workspace; JSD says nothing then).  The walk
// over the decisions already made comes first; where all children of the last node are rejected, the first one is
// evaluated once more for its residual and the draw.
template <typename LT, int NP, bool PLAIN, bool JSD>
__global__ __launch_bounds__(SNT) void trees_sequential(SequentialArgs a) {
    using RP = RawPair<LT>;
    using Raw = typename RP::raw;
    constexpr bool RES = NP > 0;
    constexpr int U = RES ? NP : 4;       // steps whose loads are in flight together
    __shared__ SeqShared sh;
    extern __shared__ __align__(16) double seq_cur[];

    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // its part of the vocabulary in scalar registers
    const int b = blockIdx.x;
    const int V = a.V;
    const int k = a.k;
    const int M = a.M;
    const int64_t c0 = (int64_t)b * M;
    const int32_t* par = a.parent + c0;
    int32_t* path = a.out_path + c0;
    // t_j(x) = max(0, cur[x]) * inv_st,  g(x) = g[x] * inv_sg
    double* cur_mem = a.work + (int64_t)b * 2 * V;
    double* g_mem = cur_mem + V;
    auto cur_at = [&](int x) { return fmax(RES ? seq_cur[x] : cur_mem[x], 0.0); };
    auto cur_set = [&](int x, double v) {
        if (RES) seq_cur[x] = v;
        else cur_mem[x] = v;
    };
    // a pair that may end beyond the vocabulary; x even and below V
    auto get2 = [&](const double* v, int x) {
        d2 r;
        if (x + 1 < V) r = *reinterpret_cast<const d2*>(v + x);
        else r = d2{v[x], 0.0};
        return r;
    };
    auto put2 = [&](double* v, int x, double lo, double hi) {
        if (x + 1 < V) *reinterpret_cast<d2*>(v + x) = d2{lo, hi};
        else v[x] = lo;
    };
    double* cur = RES ? seq_cur : cur_mem;
    // the two rows' pairs of every step, then (NP > 0) the drafter's two terms of the step in their room
    u2 tr[U], gr[U];
    const unsigned char* tab = reinterpret_cast<const unsigned char*>(sh.tab);
    double inv_st = 0.0, inv_sg = 0.0, st = 0.0, mxg = 0.0;
    auto term = [&](float l, double max) { return exp_units_nonpos((double)l - max, tab); };
    const double delta = (double)a.delta;

    // the part of the vocabulary of this wavefront: [x0, x1), in steps of a pair per lane
    const int per = ((V + SNW - 1) / SNW + PAIR_STEP - 1) / PAIR_STEP * PAIR_STEP;
    const int x0 = min(V, wave * per);
    const int x1 = min(V, x0 + per);

    const bool staged = !PLAIN && M <= SNODES;
    for (int j = tid; j < EXP_FINE_N; j += SNT) {
        sh.tab[2 * j] = EXP_FINE[2 * j] + ((uint64_t)j << 44);   // whole: exp_units_nonpos adds the exponent alone
        sh.tab[2 * j + 1] = EXP_FINE[2 * j + 1];
    }
    int first = -1;                      // PLAIN: the child whose draw is wanted
    if (PLAIN) {
        if (wave == 0) {
            int walked;
            const int found = walk_tree(a.accept + c0, nullptr, par, M, b, path, &walked);
            for (int j = walked + lane; j < M; j += WAVE) path[j] = -1;
            if (lane == 0) {
                a.out_len[b] = walked;
                sh.drawn = found;
            }
        }
        __syncthreads();
        first = sh.drawn;
        if (first < 0) {                 // uniform: nothing to draw
            if (tid == 0) a.out_next[b] = first;
            return;
        }
        first -= b * M;
    } else {
        int malformed = 0;
        for (int j = tid; j < M; j += SNT) {
            path[j] = -1;
            const int p = par[j];
            if (p < -1 || p >= j) malformed = 1;
            if (staged) {
                sh.parent[j] = p;
                sh.row[j] = a.row_index ? a.row_index[c0 + j] : (int)(c0 + j);
                sh.token[j] = a.tokens[c0 + j];
                sh.accept[j] = a.accept[c0 + j];
                sh.u_acc[j] = a.uniforms[2 * (c0 + j)];
                sh.u_res[j] = a.uniforms[2 * (c0 + j) + 1];
            }
        }
        malformed = block_or_i<SNW>(malformed, sh.ired, tid);   // its barriers publish what is staged
        if (malformed) {
            if (tid == 0) {
                a.out_len[b] = 0;
                a.out_next[b] = -3;
            }
            return;
        }
    }

    int node = -1, len = 0, next = -1;
    for (;;) {   // one sibling group per round; every branch below is uniform over the workgroup
        next = -1;
        int taken = -1;
        int group_row = -1;
        bool have_rows = false;
        const LT* grow = nullptr;
        double zz = 0.0;             // of the last rejected child: mass of what its draw is taken from,
        float u_res = 0.f;           //   its draw,
        bool zero_resid = false;     //   and whether that is the distorted target itself
        int i = node;
        for (;;) {
            if (PLAIN) {
                i = first;
            } else {
                // the next child: the smallest index above i whose parent is the node
                int child = INT_MAX;
                for (int base = i + 1; base < M; base += WAVE) {
                    const int q = base + lane;
                    const int p = q < M ? (staged ? sh.parent[q] : par[q]) : INT_MIN;
                    const unsigned long long m = __ballot(p == node);
                    if (m) {
                        child = base + __ffsll((long long)m) - 1;
                        break;
                    }
                }
                i = child;
                if (i == INT_MAX) break;
            }
            const int64_t c = c0 + i;
            const int r = staged ? sh.row[i] : a.row_index ? a.row_index[c] : (int)c;
            const int xt = staged ? sh.token[i] : a.tokens[c];
            bool usable = (unsigned)xt < (unsigned)V;
            const int32_t* nrow = a.knn + (int64_t)(usable ? xt : 0) * k;
            float u_acc32 = 0.f, u_res32 = 0.f;               // PLAIN: in flight during the passes as well
            if (PLAIN) {
                u_acc32 = a.uniforms[2 * c];
                u_res32 = a.uniforms[2 * c + 1];
            }
            int nb;
            if (!have_rows) {
                // The first child is tested against t_1 = t itself, which is the plain verification the
                // row-parallel pass has already decided for every candidate: an accepted first child is
                // taken without building the group's vectors.
                const int decided = PLAIN ? 0 : staged ? sh.accept[i] : a.accept[c];
                if (decided == 1) {
                    taken = i;
                    break;
                }
                if (decided < 0 || r < 0 || r >= a.R) {   // unusable row, token or table entry
                    next = -2;
                    break;
                }
                // rejected: the first child brings the group's rows, and is verified again below in
                // fp64 for its distorted target and residual
                nb = nrow[min(tid, k - 1)];               // in flight during the passes over the rows
                have_rows = true;
                group_row = r;
                const LT* trow = reinterpret_cast<const LT*>(a.target) + (int64_t)r * a.stride;
                grow = reinterpret_cast<const LT*>(a.draft) + (int64_t)r * a.stride;
                // Unnormalised softmax terms exp(l - max) and their sums.  A pair's load is moved to
                // the row's last two logits where it would leave the row (V = 1 reads the one logit twice).
                const int l2 = opaque_int(2 * lane);
                float mt = neg_inf_f(), mg = neg_inf_f();
                int bad = 0;
                const float inf = __builtin_huge_valf();
                auto load = [&](int xb) {
                    Raw t[U], g[U];
                    if (V == 1) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            t[u] = RP::twice(trow);
                            g[u] = RP::twice(grow);
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int x = min(xb + u * PAIR_STEP + l2, V - 2);
                            t[u] = *reinterpret_cast<const Raw*>(trow + x);
                            g[u] = *reinterpret_cast<const Raw*>(grow + x);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        tr[u] = RP::words(t[u]);
                        gr[u] = RP::words(g[u]);
                    }
                };
                auto logits = [&](u2 v, int x, float* lo, float* hi) {
                    *lo = x < x1 ? (x + 1 < V ? lo_of(v) : hi_of(v)) : neg_inf_f();
                    *hi = x + 1 < x1 ? hi_of(v) : neg_inf_f();
                };
                for (int xb = x0; xb < (RES ? x0 + 1 : x1); xb += U * PAIR_STEP) {
                    load(xb);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        // every pair lies inside the row, moved or not: no bounds in this pass
                        const float l0 = lo_of(tr[u]), l1 = hi_of(tr[u]), h0 = lo_of(gr[u]), h1 = hi_of(gr[u]);
                        if (__builtin_isunordered(l0, l1) || __builtin_isunordered(h0, h1)) bad = 1;
                        mt = fmaxf(mt, fmaxf(l0, l1));
                        mg = fmaxf(mg, fmaxf(h0, h1));
                    }
                }
                if (mt == inf || mg == inf) bad = 1;
                mt = wave_max(mt);
                mg = wave_max(mg);
                bad = wave_or(bad);
                if (lane == 0) {
                    sh.mt[wave] = mt;
                    sh.mg[wave] = mg;
                    sh.bad[wave] = bad;
                }
                __syncthreads();
                bad = 0;
                mt = mg = neg_inf_f();
#pragma unroll 4
                for (int w = 0; w < SNW; ++w) {
                    mt = fmaxf(mt, sh.mt[w]);
                    mg = fmaxf(mg, sh.mg[w]);
                    bad |= sh.bad[w];
                }
                if (bad || mt == -inf || mg == -inf) {   // uniform
                    next = -2;
                    break;
                }
                const double mxt = uniform_d((double)mt);
                mxg = uniform_d((double)mg);
                double zt = 0.0, zg = 0.0;
                // Some steps a turn, the registers moved down behind them and what comes of them put at the
                // end (NP > 0: after the last turn every step is back in its place): unrolled in full, this is
                // code that a group runs once, and fetching it costs more than the moves.
                constexpr int TURN = 2;
                for (int xb = x0; xb < (RES ? x0 + 1 : x1); xb += U * PAIR_STEP) {
                    if (!RES) load(xb);
#pragma unroll 1
                    for (int xc = xb; xc < xb + U * PAIR_STEP; xc += TURN * PAIR_STEP) {
                        u2 t2[TURN], g2[TURN];
#pragma unroll
                        for (int u = 0; u < TURN; ++u) {
                            t2[u] = g2[u] = u2{0u, 0u};
                            if (xc + u * PAIR_STEP < x1) {   // uniform over the wavefront
                                const int x = xc + u * PAIR_STEP + l2;
                                float l0 = lo_of(tr[u]), l1 = hi_of(tr[u]), h0 = lo_of(gr[u]), h1 = hi_of(gr[u]);
                                const bool whole = xc + (u + 1) * PAIR_STEP <= x1;
                                if (!whole) {
                                    logits(tr[u], x, &l0, &l1);
                                    logits(gr[u], x, &h0, &h1);
                                }
                                const double t0 = term(l0, mxt), t1 = term(l1, mxt);
                                const double g0 = term(h0, mxg), g1 = term(h1, mxg);
                                zt += t0 + t1;
                                zg += g0 + g1;
                                if (whole) *reinterpret_cast<d2*>(cur + x) = d2{t0, t1};
                                else if (x < x1) put2(cur, x, t0, t1);
                                if (!RES && x < x1) put2(g_mem, x, g0, g1);
                                t2[u] = words_of(g0);
                                g2[u] = words_of(g1);
                                asm volatile("" : "+v"(zt), "+v"(zg));   // step by step: more terms at once do not fit the registers
                            }
                        }
#pragma unroll
                        for (int u = 0; u + TURN < U; ++u) {
                            tr[u] = tr[u + TURN];
                            gr[u] = gr[u + TURN];
                        }
                        if (RES) {
#pragma unroll
                            for (int u = 0; u < TURN; ++u) {
                                tr[U - TURN + u] = t2[u];
                                gr[U - TURN + u] = g2[u];
                            }
                        }
                    }
                }
                zt = wave_sum(zt);
                zg = wave_sum(zg);
                if (lane == 0) {
                    sh.sum_a[wave] = zt;
                    sh.sum_b[wave] = zg;
                }
                __syncthreads();   // the sums, and the current target
                st = 0.0;
                double sg = 0.0;
#pragma unroll 4
                for (int w = 0; w < SNW; ++w) {
                    st += sh.sum_a[w];
                    sg += sh.sum_b[w];
                }
                st = uniform_d(st);
                inv_st = uniform_d(1.0 / st);
                inv_sg = uniform_d(1.0 / sg);
                __syncthreads();   // the walk below writes the same arrays
            } else {
                nb = nrow[min(tid, k - 1)];
            }
            if (r != group_row) usable = false;
            if (!usable) {
                next = -2;
                break;
            }

            // ---- nearest-first walk on t_j (Algorithm 2, inference part) ----
            const double gx = uniform_d(term(Lane<LT>::glob(grow, xt), mxg) * inv_sg);
            const double t_tok = uniform_d(cur_at(xt) * inv_st);
            double carry = 0.0, S = 0.0;
            int a_size = k;
            int off = 0;
            for (int j = SNT + tid; j < k; j += SNT)      // entries the walk may never reach count too
                if ((unsigned)nrow[j] >= (unsigned)V) off = 1;
            for (int base = 0; base < k; base += SNT) {
                const int j = base + tid;
                const bool valid = j < k;
                int n = base == 0 ? nb : valid ? nrow[j] : xt;
                if (!valid) n = xt;
                if ((unsigned)n >= (unsigned)V) {
                    off = 1;
                    n = xt;
                }
                const bool self = (n == xt);
                const double incl_w = wave_scan_incl(self ? 0.0 : cur_at(n) * inv_st);
                const unsigned long long any_off = __ballot(off != 0);
                if (lane == WAVE - 1) {
                    sh.sum_a[wave] = incl_w;
                    sh.bad[wave] = any_off != 0;
                }
                __syncthreads();
                double before = 0.0, ctot = 0.0;
                int bad = 0;
#pragma unroll 4
                for (int w = 0; w < SNW; ++w) {
                    if (w == wave) before = ctot;
                    ctot += sh.sum_a[w];
                    bad |= sh.bad[w];
                }
                if (bad) {   // uniform
                    usable = false;
                    break;
                }
                const double incl = carry + (before + incl_w);
                const unsigned long long failing =
                    __ballot(!self && (JSD && (!PLAIN || a.divergence) ? jsd_fails(t_tok, incl, delta) : !(incl < delta)));
                const int l = failing ? __ffsll((long long)failing) - 1 : 0;
                const double up_to = l ? __shfl(incl, l > 0 ? l - 1 : 0, WAVE) : carry + before;
                if (lane == 0) {
                    sh.cut[wave] = failing ? base + wave * WAVE + l : INT_MAX;
                    sh.sum_b[wave] = up_to;               // the sum before the failing slot
                }
                __syncthreads();
                int first = INT_MAX;
#pragma unroll 4
                for (int w = SNW - 1; w >= 0; --w)
                    if (sh.cut[w] != INT_MAX) {
                        first = sh.cut[w];
                        S = sh.sum_b[w];
                    }
                if (first != INT_MAX) {
                    a_size = first;
                    break;
                }
                carry += ctot;
                S = carry;
            }
            if (!usable) {
                next = -2;
                break;
            }
            const double mass = uniform_d(t_tok + S);
            const double u_acc = (double)(PLAIN ? u_acc32 : staged ? sh.u_acc[i] : a.uniforms[2 * c]);
            if (u_acc * gx < mass) {
                if (PLAIN) have_rows = false;   // nothing to draw from (the decision is made elsewhere)
                else taken = i;
                break;
            }

            // ---- rejected: distorted target in place, then its residual t_{j+1} ----
            // (the walk's last barrier follows every read of t_j)
            for (int j = tid; j < a_size; j += SNT) {
                const int n = j < SNT ? nb : nrow[j];
                if (n != xt) cur_set(n, 0.0);
            }
            if (tid == 0) cur_set(xt, mass * st);
            __syncthreads();
            double pr = 0.0, pt = 0.0;
            const int l2 = opaque_int(2 * lane);
            for (int xb = x0; xb < (RES ? x0 + 1 : x1); xb += U * PAIR_STEP) {
                d2 cv[U], gv[U];
                if (!RES) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int x = xb + u * PAIR_STEP + l2;
                        cv[u] = x < x1 ? get2(cur, x) : d2{0.0, 0.0};
                        gv[u] = x < x1 ? get2(g_mem, x) : d2{0.0, 0.0};
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (xb + u * PAIR_STEP < x1) {       // uniform over the wavefront
                        const int x = xb + u * PAIR_STEP + l2;
                        if (x < x1) {
                            const d2 ta = RES ? get2(cur, x) : cv[u];
                            const double g0 = RES ? double_of(tr[u]) : gv[u].x;
                            const double g1 = RES ? double_of(gr[u]) : gv[u].y;
                            const double t0 = fmax(ta.x, 0.0) * inv_st, t1 = fmax(ta.y, 0.0) * inv_st;
                            const double r0 = t0 - g0 * inv_sg, r1 = t1 - g1 * inv_sg;
                            pt += t0 + t1;
                            pr += fmax(r0, 0.0) + fmax(r1, 0.0);
                            put2(cur, x, r0 > 0.0 ? r0 : -t0, r1 > 0.0 ? r1 : -t1);
                        }
                    }
                }
            }
            pr = wave_sum(pr);
            pt = wave_sum(pt);
            if (lane == 0) {
                sh.wr[wave] = pr;
                sh.wt[wave] = pt;
            }
            __syncthreads();
            double z = 0.0, zt = 0.0;
#pragma unroll 4
            for (int w = 0; w < SNW; ++w) {
                z += sh.wr[w];
                zt += sh.wt[w];
            }
            zero_resid = !(z > 0.0);   // the residual has no mass: the distorted target is sampled
            if (zero_resid) {          // uniform; it is what the pass left, with the sign turned
                for (int x = x0 + lane; x < x1; x += WAVE) cur_set(x, fabs(cur[x]));
                __syncthreads();
            }
            zz = zero_resid ? zt : z;
            zz = uniform_d(zz);
            st = zz;
            inv_st = uniform_d(1.0 / zz);
            u_res = PLAIN ? u_res32 : staged ? sh.u_res[i] : a.uniforms[2 * c + 1];
            if (PLAIN) break;
        }
        if (taken < 0) {
            // next: -1 no child, -2 unusable; with every child rejected, the draw of the last one: the
            // first token at which the cumulative sum of t_{j+1} exceeds u times its mass
            if (next == -1 && have_rows) {
                const double* part = zero_resid ? sh.wt : sh.wr;
                const double edge = (double)u_res * zz;
                double run = 0.0, before = 0.0;
                int owner = -1, last = -1;
#pragma unroll 4
                for (int w = 0; w < SNW; ++w) {
                    const double p = part[w];
                    if (p > 0.0) {
                        if (owner < 0) {
                            last = w;
                            before = run;
                        }
                        if (owner < 0 && run + p > edge) owner = w;
                    }
                    run += p;
                }
                if (owner < 0) owner = last;   // rounding left no crossing: the last part with mass
                if (owner < 0) break;          // no mass at all (sums that are not numbers): next stays -1
                if (wave == owner) {
                    int found = -1, last_pos = -1;
                    const int l2 = opaque_int(2 * lane);
                    for (int xb = x0; xb < x1 && found < 0; xb += PAIR_STEP) {
                        const int x = xb + l2;
                        const d2 v = x < x1 ? get2(cur, x) : d2{0.0, 0.0};
                        const double r0 = fmax(v.x, 0.0), r1 = fmax(v.y, 0.0);
                        const double own = r0 + r1;
                        const double incl = before + wave_scan_incl(own);
                        const unsigned long long cross = __ballot(own > 0.0 && incl > edge);
                        const unsigned long long has = __ballot(own > 0.0);
                        const bool first = r0 > 0.0 && (!(r1 > 0.0) || incl - r1 > edge);
                        if (cross) found = __shfl(first ? x : x + 1, __ffsll((long long)cross) - 1, WAVE);
                        if (has) last_pos = __shfl(r1 > 0.0 ? x + 1 : x, 63 - __clzll((long long)has), WAVE);
                        before = lane63_d(incl);
                    }
                    if (lane == 0) sh.drawn = found >= 0 ? found : last_pos;
                }
                __syncthreads();
                next = sh.drawn;
            }
            break;
        }
        if (tid == 0) path[len] = taken;
        len += 1;
        node = taken;
    }
    if (tid == 0) {
        if (!PLAIN) a.out_len[b] = len;
        a.out_next[b] = next;
    }
}

// The current target in LDS and the drafter's terms in registers as long as V doubles fit beside the
// kernel's static data: up to 19200 tokens; instantiations of 2, 8 and 10 steps per wavefront, because a
// step beyond the vocabulary still loads (from a clamped address) and holds four registers per lane.
constexpr int SEQ_LDS_MAX_V = 150 * 1024 / (int)sizeof(double);
static_assert(SNW * 10 * PAIR_STEP >= SEQ_LDS_MAX_V, "ten steps cover what fits in LDS");
static_assert(SEQ_LDS_MAX_V * sizeof(double) + sizeof(SeqShared) <= 160 * 1024, "LDS of a workgroup");

template <typename LT, int NP, bool PLAIN, bool JSD>
static hipError_t launch_steps(const SequentialArgs& a, hipStream_t stream, bool launch) {
    const size_t lds = NP > 0 ? (size_t)a.V * sizeof(double) : 0;
    const hipError_t e = allow_lds<&trees_sequential<LT, NP, PLAIN, JSD>>(lds);
    if (e != hipSuccess || !launch) return e;
    hipLaunchKernelGGL((trees_sequential<LT, NP, PLAIN, JSD>), dim3(a.B), dim3(SNT), lds, stream, a);
    return hipGetLastError();
}

template <typename LT, bool PLAIN, bool JSD>
static hipError_t launch_bound(const SequentialArgs& a, hipStream_t stream, bool launch) {
    if (a.V <= SNW * 2 * PAIR_STEP) return launch_steps<LT, 2, PLAIN, JSD>(a, stream, launch);
    if (a.V <= SNW * 8 * PAIR_STEP) return launch_steps<LT, 8, PLAIN, JSD>(a, stream, launch);
    if (a.V <= SEQ_LDS_MAX_V) return launch_steps<LT, 10, PLAIN, JSD>(a, stream, launch);
    if constexpr (PLAIN) return hipErrorInvalidValue;   // tree_plain_fits tells
    else return launch_steps<LT, 0, false, JSD>(a, stream, launch);
}

// A kernel for each bound on the neighbourhood: see the top of the file.
template <typename LT, bool PLAIN>
static hipError_t launch_typed(const SequentialArgs& a, hipStream_t stream, bool launch) {
    if constexpr (PLAIN) {
        return launch_bound<LT, true, true>(a, stream, launch);   // no loop over groups: registers to spare
    } else {
        if (launch) return a.divergence ? launch_bound<LT, false, true>(a, stream, true) : launch_bound<LT, false, false>(a, stream, true);
        const hipError_t e = launch_bound<LT, false, false>(a, stream, false);
        return e == hipSuccess ? launch_bound<LT, false, true>(a, stream, false) : e;
    }
}

// Loads the kernels on the current device and raises their LDS limit for this vocabulary size.
hipError_t prepare_sequential(int logits_dtype, int V) {
    SequentialArgs a{};
    a.V = V;
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, logits_dtype == 0
                                                   ? reinterpret_cast<const void*>(&trees_sequential<float, 0, false, false>)
                                                   : reinterpret_cast<const void*>(&trees_sequential<uint16_t, 0, false, false>));
    if (e != hipSuccess) return e;
    e = logits_dtype == 0 ? launch_typed<float, false>(a, nullptr, false) : launch_typed<uint16_t, false>(a, nullptr, false);
    if (e == hipSuccess && tree_plain_fits(V))
        e = logits_dtype == 0 ? launch_typed<float, true>(a, nullptr, false) : launch_typed<uint16_t, true>(a, nullptr, false);
    return e;
}

hipError_t launch_trees_sequential(const SequentialArgs& a, int logits_dtype, hipStream_t stream) {
    return logits_dtype == 0 ? launch_typed<float, false>(a, stream, true) : launch_typed<uint16_t, false>(a, stream, true);
}

bool tree_plain_fits(int V) { return V <= SEQ_LDS_MAX_V; }

hipError_t launch_trees_plain(const SequentialArgs& a, int logits_dtype, hipStream_t stream) {
    return logits_dtype == 0 ? launch_typed<float, true>(a, stream, true) : launch_typed<uint16_t, true>(a, stream, true);
}

}  // namespace lantern
