// sa_draw.h -- e^x and the draws of a variable whose energy is linear in its value, one lane each: by the
// inverse of the distribution (linear_draw) and in closed form (heat_bath_closed).  Nothing here needs a wave:
// tests/draw_bounds.cpp compiles it for the host, with the gfx950 builtins by their host counterparts.
#pragma once

#include <cstdint>

namespace sa {
namespace {

// e^x for x <= 0 (every exponential of the annealer has a non-positive argument): x = n ln 2 + r
// with |r| <= ln(2)/2, e^r by the degree-11 polynomial that interpolates it at the 12 Chebyshev
// nodes of that interval (relative error below 2^-55.7; gen_exp_poly.py derives the coefficients
// and checks the routine: at most about 0.83 ulp), then scaled by 2^n.  The scaling rounds once,
// so below -745.2, where e^x is under half the smallest subnormal, the result is 0 (arguments
// under -746 are clamped there first).  Within about an ulp, like the host library the oracle
// uses; a last-bit difference moves a draw only when a uniform number falls within that ulp of a
// threshold.
__device__ __forceinline__ double exp_nonpos(double x) {
    const double xc = x > -746.0 ? x : -746.0;
    const double n = rint(xc * 1.4426950408889634);     // 1 / ln 2
    double r = fma(-n, 0.6931471803691238, xc);          // ln 2 rounded to 32 bits (n * it exact)
    r = fma(-n, 1.9082149292705877e-10, r);              // the rest of ln 2
    double p = 2.5110037605963777e-08;
    p = fma(p, r, 2.763263963904103e-07);
    p = fma(p, r, 2.755724091857897e-06);
    p = fma(p, r, 2.4801485482328494e-05);
    p = fma(p, r, 0.00019841269890047113);
    p = fma(p, r, 0.0013888888952314775);
    p = fma(p, r, 0.008333333333319601);
    p = fma(p, r, 0.0416666666664881);
    p = fma(p, r, 0.1666666666666668);
    p = fma(p, r, 0.5000000000000019);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_amdgcn_ldexp(p, (int)n);
}

// expm1(x) for x <= 0 (the closed-form heat bath's expm1(-c W)).  Below -40, e^x is under half an
// ulp of 1 and the value is -1 exactly.  On [-0.35, 0] the Taylor series of e^x - 1 to x^14 (error
// below 2^-60 relative); otherwise e^x - 1, which cancels nothing because e^x <= 0.71.
__device__ __forceinline__ double expm1_nonpos(double x) {
    if (x < -40.0) return -1.0;
    if (x < -0.35) return exp_nonpos(x) - 1.0;
    // Horner on 1/k!, k = 14 .. 2, then x + x^2 (...)
    double p = 1.0 / 87178291200.0;            // 1/14!
    p = fma(p, x, 1.0 / 6227020800.0);         // 1/13!
    p = fma(p, x, 1.0 / 479001600.0);          // 1/12!
    p = fma(p, x, 1.0 / 39916800.0);           // 1/11!
    p = fma(p, x, 1.0 / 3628800.0);            // 1/10!
    p = fma(p, x, 1.0 / 362880.0);             // 1/9!
    p = fma(p, x, 1.0 / 40320.0);              // 1/8!
    p = fma(p, x, 1.0 / 5040.0);               // 1/7!
    p = fma(p, x, 1.0 / 720.0);                // 1/6!
    p = fma(p, x, 1.0 / 120.0);                // 1/5!
    p = fma(p, x, 1.0 / 24.0);                 // 1/4!
    p = fma(p, x, 1.0 / 6.0);                  // 1/3!
    p = fma(p, x, 0.5);                        // 1/2!
    return fma(p * x, x, x);
}

// log1p(y) for -1 < y <= 0 (the closed-form heat bath's log1p(U m)).  u = 1 + y rounded; log(u)
// from u = f 2^e with f in [sqrt(1/2), sqrt(2)) and log f = 2 atanh(s), s = (f - 1)/(f + 1),
// |s| <= 0.1716, by its odd series to s^21 (error below 2^-62 relative); the rounding of u is
// put back to first order, log1p(y) = log(u) + (y - (u - 1)) / u (Kahan's correction).
__device__ __forceinline__ double log1p_nonpos(double y) {
    if (y == 0.0) return 0.0;
    if (y <= -1.0) return -__builtin_huge_val();
    const double u = 1.0 + y;
    const double corr = (y - (u - 1.0)) * __builtin_amdgcn_rcp(u);
    int e = __builtin_amdgcn_frexp_exp(u);
    double f = __builtin_amdgcn_frexp_mant(u);  // [0.5, 1)
    if (f < 0.70710678118654752) {
        f = f + f;
        e -= 1;
    }
    const double s = (f - 1.0) / (f + 1.0);
    const double s2 = s * s;
    double r = 1.0 / 21.0;
    r = fma(r, s2, 1.0 / 19.0);
    r = fma(r, s2, 1.0 / 17.0);
    r = fma(r, s2, 1.0 / 15.0);
    r = fma(r, s2, 1.0 / 13.0);
    r = fma(r, s2, 1.0 / 11.0);
    r = fma(r, s2, 1.0 / 9.0);
    r = fma(r, s2, 1.0 / 7.0);
    r = fma(r, s2, 1.0 / 5.0);
    r = fma(r, s2, 1.0 / 3.0);
    const double ln2_hi = 0.6931471803691238;    // ln 2 rounded to 32 bits: e * ln2_hi is exact
    const double ln2_lo = 1.9082149292705877e-10;  // ln 2 - ln2_hi
    const double ed = (double)e;
    const double two_s = s + s;
    // log u = e ln2_hi + (2 s + (2 s s^2 r + e ln2_lo)) + corr
    return fma(ed, ln2_hi, two_s + (fma(two_s * s2, r, ed * ln2_lo) + corr));
}

// Cumulative weights in value order, by one lane: the value drawn where the closed form cannot tell.
// Values 746 / c and further from the end of least energy weigh exactly 0 (exp_nonpos) and are passed over.
__device__ __forceinline__ uint32_t linear_draw_by_sums(bool from_top, double slope, uint32_t W, double beta, double U) {
    const double reach = 746.0 / (beta * slope) + 2.0;   // (beta slope > 0; infinite or beyond W: every value)
    const uint32_t m = reach < (double)W ? (uint32_t)reach + 1u : W;
    const uint32_t n = m < W ? m : W, j0 = from_top ? W - n : 0u;
    double total = 0.0;
    for (uint32_t i = 0; i < n; ++i) total += exp_nonpos(-(beta * (slope * (double)(from_top ? n - 1u - i : i))));
    const double thr = U * total;
    double run = 0.0;
    for (uint32_t i = 0; i < n; ++i) {
        run += exp_nonpos(-(beta * (slope * (double)(from_top ? n - 1u - i : i))));
        if (run > thr) return j0 + i;
    }
    return W - 1u;
}

// The closed form in double precision; false where it cannot tell.  With y = P m and u = 1 + y (P, m below), m
// and y are rounded to some 2^-53 of themselves, which is y / u of log1p(y) and so y / (u c) of x: small
// except in the tail, where u may be as small as 2^-53.  log1p, the division and c add some ulp of x <= W.
// So a step within 1e-10 + 1e-14 W + 1e-15 |y| / (u c) is left to the sums (of 3,000,000 draws, most of
// them at steps, none that was decided left the value of 113-bit arithmetic, also with a tenth of this margin),
// and so is u = 0 (U = 0 drawn from the top).
__device__ __forceinline__ bool linear_draw_double(bool from_top, double slope, uint32_t W, double beta, double U, uint32_t &j) {
    const double c = beta * slope, Wd = (double)W;
    const double m = expm1_nonpos(-(c * Wd));
    const double y = (from_top ? 1.0 - U : U) * m, u = 1.0 + y;
    const double L = log1p_nonpos(y) / c;
    const double x = from_top ? Wd + L : -L;
    const double near = rint(x), tol = 1e-10 + 1e-14 * Wd - 1e-15 * (y / u) / c;
    // (steps 0 and W decide nothing; a NaN fails)
    if (!(u > 0.0 && tol < 0.25)) return false;
    if (!(__builtin_fabs(x - near) > tol) && near > 0.5 && near < Wd - 0.5) return false;
    j = !(x > 0.0) ? 0u : x >= Wd ? W - 1u : (uint32_t)ceil(x) - 1u;
    return true;
}

// In single precision: m from the series of expm1 (c W < 1/2; the first term left out is 3.9e-6 of m at
// 1/2, rounding 4e-7) or e^-cW - 1 (below 1e-6 as |m| > 0.39); y = P m to 5e-6, from the exponential 1.2e-6;
// log1p(y) from the series of 2 atanh(y / (2 + y)) (|y| < 0.3, where log1p passes on at most 1.2 of y's
// relative error: 6e-6 in all) or log(1 + y), off by that of y times |y| / (1 + y), at most 3e-6, and by 1e-6 of
// itself; 1 / c, the product and W - x by 3e-7 W.  `err` is at least 1.6 times that (2.5 times the
// largest of 2,000,000 errors, with correctly rounded exp2, log2 and reciprocal).
__device__ __forceinline__ void linear_draw_single(bool from_top, double c, uint32_t W, double U, float &x, float &err) {
    const float cf = (float)c, Wf = (float)W;
    const float t = cf * Wf;
    const float series = -t * (1.0f - t * (0.5f - t * (0.16666667f - t * (0.041666667f - t * (0.0083333333f - t * 0.0013888889f)))));
    const float m = t < 0.5f ? series : __builtin_amdgcn_exp2f(t * -1.4426950f) - 1.0f;
    const float y = (float)(from_top ? 1.0 - U : U) * m;
    const float s = y * __builtin_amdgcn_rcpf(2.0f + y), s2 = s * s;
    const float near0 = 2.0f * s * (1.0f + s2 * (0.33333333f + s2 * (0.2f + s2 * (0.14285714f + s2 * 0.11111111f))));
    const float u = 1.0f + y;
    const bool small = y > -0.3f;
    const float L = small ? near0 : __builtin_amdgcn_logf(u) * 0.69314718f;
    const float ic = __builtin_amdgcn_rcpf(cf);
    const float aL = -L;
    err = (small ? 1e-5f * aL : 5e-6f * __builtin_amdgcn_rcpf(u) + 4e-6f * aL) * ic + 1e-6f * Wf;
    x = from_top ? Wf - aL * ic : aL * ic;
}

// The index drawn where single precision cannot tell.
__device__ __forceinline__ uint32_t linear_draw_rest(bool from_top, double slope, uint32_t W, double beta, double U) {
    uint32_t i;
    if (!(beta * slope > 1e-280)) {   // every weight is 1: the count of v - l + 1 <= U W
        i = (uint32_t)(U * (double)W);
        return i < W ? i : W - 1u;
    }
    if (!linear_draw_double(from_top, slope, W, beta, U, i)) i = linear_draw_by_sums(from_top, slope, W, beta, U);
    return i;
}
// The same out of line (kApart below): its registers are then not the caller's.
__device__ __attribute__((noinline, unused)) uint32_t linear_draw_rest_apart(bool from_top, double slope, uint32_t W,
                                                                             double beta, double U) {
    return linear_draw_rest(from_top, slope, W, beta, U);
}

// Heat-bath draw of a variable with dE(v) = a (v - z_k): the first value whose cumulative weight exceeds
// U times the total.  Index i = ceil(x) - 1 with x = -log1p(P m) / c from the lower end for a > 0, W + the
// same for a < 0; c = beta |a|, m = expm1(-c W), P = U or 1 - U.
//
// It replaced the enumeration in every kernel: 32 random-interaction problems (N = 100, W = 201, most
// variables linear; 100 sweeps x 100 reads) 24.6 to 20.1 ms, 64 mixed problems 103 to 95 ms.
template <bool kApart = false>
__device__ __forceinline__ int64_t linear_draw(int64_t a, int64_t lo, uint32_t W, double beta, double U) {
    const bool from_top = a < 0;
    const double slope = (double)(from_top ? -a : a);
    const double c = beta * slope;
    float x, err;
    linear_draw_single(from_top, c, W, U, x, err);
    const float Wf = (float)W, step = __builtin_rintf(x);
    // a NaN or an infinity anywhere (c = 0, 1 + y = 0) fails the comparison; steps 0 and W decide nothing
    const bool sure = W < (1u << 20) && err < 0.25f &&
                      (__builtin_fabsf(x - step) > err || step < 0.5f || step > Wf - 0.5f) && c > 1e-30;
    uint32_t i = x <= 0.0f ? 0u : (uint32_t)__builtin_ceilf(x) - 1u;
    i = i < W ? i : W - 1u;
    if (!sure)
        i = kApart ? linear_draw_rest_apart(from_top, slope, W, beta, U) : linear_draw_rest(from_top, slope, W, beta, U);
    return lo + (int64_t)i;
}

// Heat bath for a variable whose energy difference is linear, dE(v) = a (v - z_k) (Sec. 3.3.2,
// multilinear case): the inverse of the cumulative distribution in O(1).  Index i = v - lo has
// probability proportional to exp(-beta a i); with c = beta |a| and g(q) = -log1p(q expm1(-c W)) / c
// the paper's x = -(T/a) ln[1 - U (1 - exp(-a W / T))] is g(U) for a > 0 and W - g(1 - U) for a < 0
// (the same value without overflowing exp(c W)); v = lo + ceil(x) - 1, clamped to the box.  a = 0
// or beta = 0 is the uniform distribution, drawn from x1 by a multiply-high.  Wave-uniform.
// expm1 and log1p are the functions above (about an ulp, like the host library); a last-bit
// difference moves a draw only when x lies within a few ulps of an integer.
__device__ __forceinline__ int64_t heat_bath_closed(int64_t a, int64_t lo, int64_t W, double beta, double U,
                                                    uint32_t x1) {
    const double c = beta * (double)(a < 0 ? -a : a);
    if (a == 0 || !(c > 0.0)) return lo + (int64_t)(((uint64_t)x1 * (uint64_t)W) >> 32);
    const double Wd = (double)W;
    const double m = expm1_nonpos(-(c * Wd));
    double x;
    if (a > 0)
        x = -log1p_nonpos(U * m) / c;
    else
        x = Wd + log1p_nonpos((1.0 - U) * m) / c;
    if (!(x > 0.0)) return lo;
    if (x >= Wd) return lo + W - 1;
    return lo + (int64_t)ceil(x) - 1;
}

// The margin of a settled sweep (sa_settled.h) as it is kept: M rounded down to the upper half of a float; 0
// where M <= 0.
__device__ __forceinline__ uint16_t margin_bits(int64_t M) {
    if (M <= 0) return 0;
    // below M after the conversion's rounding, then cut to 16 bits (toward zero)
    const float f = (float)M * 0.9999998f;
    uint32_t b;
    __builtin_memcpy(&b, &f, 4);
    return (uint16_t)(b >> 16);
}

// Whether a linear variable may be passed over without its random number once every other value's weight is
// 0. Not at the top of its range with the closed-form draw, which gives the lowest value at U = 0.
__device__ __forceinline__ bool may_freeze(bool closed, int64_t lo, int64_t zk) { return !closed || zk == lo; }

// Every value of the variable has the same energy.
constexpr uint16_t kFlat = 0x8000;
// The kept margin of a linear variable at z_k with coefficient a1; with the sign bit set where it may not freeze.
__device__ __forceinline__ uint16_t linear_margin(bool closed, int64_t a1, int64_t lo, int64_t hi, int64_t zk) {
    if (a1 == 0) return kFlat;
    const uint16_t b = margin_bits(zk == lo ? a1 : zk == hi ? -a1 : 0);
    return b != 0 && !may_freeze(closed, lo, zk) ? (uint16_t)(b | 0x8000u) : b;
}

// And of a variable that never moves.
constexpr uint16_t kFixed = 0x7FFF;
// The margins i .. i + 3 of n after a change that may have moved all of them: not known, but those past n, which
// are read with the others, stay those of variables that never move.
__device__ __forceinline__ uint64_t cleared_margins(int32_t i, int32_t n) {
    return i + 4 <= n ? 0ull : (~0ull << (16 * (n - i))) & 0x7FFF7FFF7FFF7FFFull;
}

}  // namespace
}  // namespace sa
