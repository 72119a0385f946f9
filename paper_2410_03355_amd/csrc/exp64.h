// exp(d) for d <= 0 in fp64: argument reduction by ln 2 in two pieces
// (Cody-Waite) and the degree-13 Taylor polynomial on |r| <= ln(2)/2, whose
// truncation error is below 2^-57; the result is within one ulp of libm.
// Branch-free.  The same source compiles for the device and, for testing
// against libm, for the host.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define LANTERN_HD __host__ __device__ __forceinline__
#else
#define LANTERN_HD inline
#endif

namespace lantern {

// One Horner step acc*r + c.  On the device the constant stays in a scalar
// register pair and the step is a single v_fma_f64 (the compiler otherwise
// copies the constant into the accumulator register first).
LANTERN_HD double horner_step(double acc, double r, double c) {
#if defined(__HIP_DEVICE_COMPILE__)
    double out;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(out) : "v"(acc), "v"(r), "s"(c));
    return out;
#else
    return __builtin_fma(acc, r, c);
#endif
}

// d <= 0, or -inf (result 0).  Arguments below -1000, and NaN, give 0.
LANTERN_HD double exp_nonpos(double d) {
    const double LOG2E = 1.4426950408889634074;          // 1/ln 2
    const double LN2_HI = 6.93147180369123816490e-01;    // ln 2 with the low 21 mantissa bits zero
    const double LN2_LO = 1.90821492927058770002e-10;    // ln 2 - LN2_HI
    d = fmax(d, -1000.0);                                 // 2^-1443 scales to exactly 0 below
    const double n = __builtin_rint(d * LOG2E);
    double r = __builtin_fma(-n, LN2_HI, d);
    r = __builtin_fma(-n, LN2_LO, r);
    double p = 1.6059043836821614599e-10;                 // 1/13!
    p = horner_step(p, r, 2.0876756987868098979e-09);     // 1/12!
    p = horner_step(p, r, 2.5052108385441718775e-08);     // 1/11!
    p = horner_step(p, r, 2.7557319223985890653e-07);     // 1/10!
    p = horner_step(p, r, 2.7557319223985892511e-06);     // 1/9!
    p = horner_step(p, r, 2.4801587301587301566e-05);     // 1/8!
    p = horner_step(p, r, 1.9841269841269841253e-04);     // 1/7!
    p = horner_step(p, r, 1.3888888888888889419e-03);     // 1/6!
    p = horner_step(p, r, 8.3333333333333332177e-03);     // 1/5!
    p = horner_step(p, r, 4.1666666666666664354e-02);     // 1/4!
    p = horner_step(p, r, 1.6666666666666665741e-01);     // 1/3!
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return ldexp(p, (int)n);
}

// exp(d) for d in [-1000, 700] from a table of 2^(j/128): d = (128 n + j) ln2/128 + r with
// |r| <= ln2/256, exp(d) = 2^n * T[j] * e^r.  The reduction multiplies the integer 128 n + j
// (below 2^18 in magnitude) by a 32-bit piece of ln2/128, which is exact, and by the remainder;
// e^r - 1 is the degree-5 Taylor polynomial (truncation below 6e-19); the table entry is a pair
// hi + lo, so the result is within 0.6 ulp of the exact value: within one ulp of libm.  Half the
// arithmetic of exp_nonpos.  tab: EXP_TABLE_HILO, on the device a copy of it in LDS.
// Arguments below -1000, and NaN, give 0.  Branch-free.
LANTERN_HD double exp_poly5(double r) {                     // e^r - 1 for |r| <= ln2/256
    double q = __builtin_fma(r, 8.3333333333333332177e-03, 4.1666666666666664354e-02);   // 1/5!, 1/4!
    q = __builtin_fma(q, r, 1.6666666666666665741e-01);                                  // 1/3!
    q = __builtin_fma(q, r, 0.5);
    q = __builtin_fma(q, r, 1.0);
    return q * r;
}

LANTERN_HD double exp_tab(double d, const double* tab) {
    const double INV_STEP = 184.6649652337873;             // 128 / ln 2
    const double STEP_HI = 0x1.62e42fee00000p-8;           // ln2/128 with the low 21 mantissa bits zero
    const double STEP_LO = 0x1.a39ef35793c76p-40;          // ln2/128 - STEP_HI
    d = fmin(fmax(d, -1000.0), 700.0);
    const double m = __builtin_rint(d * INV_STEP);
    double r = __builtin_fma(-m, STEP_HI, d);
    r = __builtin_fma(-m, STEP_LO, r);
    const int mi = (int)m;
    const int j = mi & 127;
    const int n = mi >> 7;                                  // floor division: j >= 0
#if defined(__HIP_DEVICE_COMPILE__)
    typedef double pair_t __attribute__((ext_vector_type(2)));
    const pair_t entry = reinterpret_cast<const pair_t*>(tab)[j];   // one 16-byte load: the table is aligned
    const double hi = entry.x, lo = entry.y;
#else
    const double hi = tab[2 * j], lo = tab[2 * j + 1];
#endif
    const double p = exp_poly5(r);                          // e^r - 1
    const double res = hi + __builtin_fma(hi, p, lo);
    return ldexp(res, n);
}

// The form that the fp64 pass over a rejected row uses: 15 instructions a value, the clamp and the conversion of its logit
// and the table's lookup among them.  Terms are counted in steps of
// ln2/256 from a whole number of steps K common to the row: e^l 2^(-K/256), with the logit l taken as it is (no
// subtraction of a reference: K only scales the terms).
//   l = m ln2/256 + r with m = rint(l 256/ln2), |r| <= ln2/512: one fused multiply-add onto 1.5 2^52 - K leaves
//   m - K in the low word of the sum; e^r - 1 is a polynomial of degree four whose cubic coefficient is raised to
//   cover the fifth-order term (error below 6e-18); the table (EXP_FINE) holds 2^(j/256) as hi (1 + rest), so the
//   remainder goes in with the polynomial, and its hi comes without the j 2^44 that (m - K) 2^44 puts back with the
//   exponent: one addition to the high word, and the value is one fused multiply-add.
// Error: half an ulp of that last step and below 0.05 ulp of the rest, for |l| <= 5600 (|m| < 2^21) and results in the
// normal range; the caller clamps: rows with a reference beyond 4096 in magnitude are not evaluated here, and no logit is
// taken more than 1100 below it.  start: EXP_UNITS_START - K.  tab_bytes: the table, 16-byte aligned; on the device an object
// of its own in LDS, whose place is known when the kernel is compiled: the lookup's address is then two instructions and
// a constant of the load, with no base to add.
constexpr double EXP_UNITS_START = 6755399441055744.0;       // 1.5 * 2^52
constexpr double EXP_UNITS_INV = 0x1.71547652b82fep+8;       // 256 / ln 2
constexpr double EXP_UNITS_HI = 0x1.62e42ff000000p-9;        // ln2/256 to 32 bits: exact times |m| < 2^21
constexpr double EXP_UNITS_LO = -0x1.718432a1b0e26p-43;      // ln2/256 - EXP_UNITS_HI
struct ExpUnits {
    unsigned mi;     // m - K, two's complement
    double hi, p;    // the value is hi (1 + p) with (m - K) 2^44 added to the bits of hi
};
LANTERN_HD ExpUnits exp_units_parts(double l, double start, const unsigned char* tab_bytes) {
    ExpUnits u;
    const double t = __builtin_fma(l, EXP_UNITS_INV, start);
    unsigned long long tb;
    __builtin_memcpy(&tb, &t, 8);
    u.mi = (unsigned)tb;
    const double m = t - start;
    double r = __builtin_fma(-m, EXP_UNITS_HI, l);
    r = __builtin_fma(-m, EXP_UNITS_LO, r);
    double rest;
    const unsigned char* at = tab_bytes + ((u.mi << 4) & 0xFF0u);
#if defined(__HIP_DEVICE_COMPILE__)
    typedef double pair_t __attribute__((ext_vector_type(2)));
    const pair_t entry = *reinterpret_cast<const pair_t*>(at);      // one 16-byte load: the table is aligned
    u.hi = entry.x;
    rest = entry.y;
#else
    __builtin_memcpy(&u.hi, at, 8);
    __builtin_memcpy(&rest, at + 8, 8);
#endif
    double q = __builtin_fma(r, 4.1666666666666664354e-02, 0.16666667995547);   // 1/24, 1/6 + 1.33e-8
    q = __builtin_fma(q, r, 0.5);
    q = __builtin_fma(q, r, 1.0);
    u.p = __builtin_fma(q, r, rest);
    return u;
}
LANTERN_HD double exp_units_scaled(double hi, unsigned steps) {   // steps 2^44 added to the bits
    unsigned long long hb;
    __builtin_memcpy(&hb, &hi, 8);
    const unsigned high = (unsigned)(hb >> 32) + (steps << 12);
    hb = ((unsigned long long)high << 32) | (unsigned)hb;
    __builtin_memcpy(&hi, &hb, 8);
    return hi;
}
LANTERN_HD double exp_units(double l, double start, const unsigned char* tab_bytes) {
    const ExpUnits u = exp_units_parts(l, start, tab_bytes);
    const double hi = exp_units_scaled(u.hi, u.mi);
    return __builtin_fma(hi, u.p, hi);
}
// e^d for d <= 0 (or -inf, result 0) from a table whose hi is whole (j 2^44 put back when it is laid out); results below
// the normal range are rounded there, in the end zero.  The clamp is on the fp64 difference that the caller forms: a floor
// in fp32 under a row's maximum is the maximum itself once that has no units left (from 2^35 on for 1100).
LANTERN_HD double exp_units_nonpos(double d, const unsigned char* tab_bytes) {
#if defined(__HIP_DEVICE_COMPILE__)
    double c;                                               // fmax would quiet its operands first
    asm("v_max_f64 %0, %1, %2" : "=v"(c) : "v"(d), "s"(-1100.0));
    d = c;
#else
    d = fmax(d, -1100.0);
#endif
    const ExpUnits u = exp_units_parts(d, EXP_UNITS_START, tab_bytes);
    return ldexp(__builtin_fma(u.hi, u.p, u.hi), (int)u.mi >> 8);
}
// exp_units for results that may lie below the normal range.
LANTERN_HD double exp_units_any(double l, double start, const unsigned char* tab_bytes) {
    const ExpUnits u = exp_units_parts(l, start, tab_bytes);
    const double hi = exp_units_scaled(u.hi, u.mi & 255u);
    return ldexp(__builtin_fma(hi, u.p, hi), (int)u.mi >> 8);
}

}  // namespace lantern
