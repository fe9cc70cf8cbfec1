// The draws of csrc/sa_draw.h compiled for the host and held against 113-bit arithmetic and against the
// cumulative weights added one by one.  argv[1] names a check; prints its figures and "ok".
#include <quadmath.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

// the gfx950 builtins' host counterparts (theirs err by an ulp, these by half)
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_logf(x) log2f(x)
#define __builtin_amdgcn_ldexp(x, n) ldexp(x, n)
static inline int frexp_exp(double x) {
    int e;
    (void)frexp(x, &e);
    return e;
}
static inline double frexp_mant(double x) {
    int e;
    return frexp(x, &e);
}
#define __builtin_amdgcn_frexp_exp(x) frexp_exp(x)
#define __builtin_amdgcn_frexp_mant(x) frexp_mant(x)
#include "../paper_2511_17245_amd/csrc/sa_draw.h"

namespace {

using Quad = __float128;
int failures = 0;
void fail(const char *what, double c, uint32_t W, bool top, double U) {
    if (failures++ < 10) std::fprintf(stderr, "FAILED: %s (c %.17g W %u from %s U %.17g)\n", what, c, W, top ? "top" : "bottom", U);
}

std::mt19937_64 g(2511);
double unit() { return (double)(g() >> 11) * 0x1p-53; }   // as the kernels form U
double log_uniform(double a, double b) { return std::exp(std::log(a) + unit() * (std::log(b) - std::log(a))); }
// U over its range, near 0 and near 1
double some_u() {
    switch (g() % 4) {
        case 0: return (double)(g() % 4096) * 0x1p-53;
        case 1: return 1.0 - (double)(1 + g() % (1ull << (g() % 40 + 1))) * 0x1p-53;
        default: return unit();
    }
}

// the inverse of the distribution
Quad exact_x(double slope, double beta, uint32_t W, bool top, double U) {
    const Quad c = (Quad)beta * (Quad)slope, m = expm1q(-c * (Quad)W);
    const Quad L = log1pq((top ? (Quad)1 - (Quad)U : (Quad)U) * m) / c;
    return top ? (Quad)W + L : -L;
}
uint32_t index_of(Quad x, uint32_t W) { return x <= 0 ? 0u : x >= (Quad)W ? W - 1u : (uint32_t)ceilq(x) - 1u; }

// U at a step of the distribution, a few units of 2^-53 to either side
double u_near_step(double slope, double beta, uint32_t W, bool top) {
    const Quad c = (Quad)beta * (Quad)slope;
    const uint32_t j = 1u + (uint32_t)(g() % (W - 1u));   // between values j - 1 and j
    Quad cum = expm1q(-c * (Quad)j) / expm1q(-c * (Quad)W);
    if (top) cum = expq(-c * (Quad)(W - j)) * cum;
    const double k = (double)rintq(cum * (Quad)0x1p53) + (double)((int)(g() % 9) - 4);
    return k < 0 ? 0.0 : k >= 0x1p53 ? 1.0 - 0x1p-53 : k * 0x1p-53;
}

uint32_t plain_sums(bool top, double slope, uint32_t W, double beta, double U) {
    std::vector<double> run((size_t)W);
    double total = 0.0;
    for (uint32_t j = 0; j < W; ++j) {
        total += sa::exp_nonpos(-(beta * (slope * (double)(top ? W - 1u - j : j))));
        run[j] = total;
    }
    for (uint32_t j = 0; j < W; ++j)
        if (run[j] > U * total) return j;
    return W - 1u;
}

// |x - exact| in single precision against the bound
void single() {
    double worst = 0.0;
    for (int i = 0; i < 2000000; ++i) {
        const uint32_t W = (uint32_t)log_uniform(2.0, (double)(1 << 20));
        const double c = i % 8 == 0 ? log_uniform(0.2, 0.5) / W : i % 2 ? log_uniform(1e-9, 1e3) / W : log_uniform(1e-6, 100.0);
        const bool top = g() % 2;
        const double U = some_u();
        float x, err;
        sa::linear_draw_single(top, c, W, U, x, err);
        if (!(err < 0.25f)) continue;   // not used
        const double d = std::fabs((double)((Quad)x - exact_x(c, 1.0, W, top, U)));
        worst = std::max(worst, d / (double)err);
        if (!(d * 1.6 <= (double)err)) fail("single precision within its bound", c, W, top, U);
    }
    std::printf("single: largest error / bound %.3f\n", worst);
}

// Where the double-precision form decides it draws the exact value: at U near steps, tails among them
void decided() {
    int64_t decided = 0, left = 0;
    for (int i = 0; i < 3000000; ++i) {
        const uint32_t W = (uint32_t)log_uniform(2.0, i % 3 ? 3000.0 : 3e6);
        const double c = i % 2 ? log_uniform(1e-4, 60.0) / W : log_uniform(1e-6, 100.0);
        const bool top = g() % 2;
        const double beta = log_uniform(1e-3, 1e3), slope = std::max(1.0, std::rint(c / beta));
        const double U = i % 4 ? u_near_step(slope, beta, W, top) : some_u();
        uint32_t j = 0;
        if (!sa::linear_draw_double(top, slope, W, beta, U, j)) {
            ++left;
            continue;
        }
        ++decided;
        if (j != index_of(exact_x(slope, beta, W, top, U), W)) fail("double precision decides as the exact inverse", beta * slope, W, top, U);
    }
    std::printf("decided %lld, left to the sums %lld\n", (long long)decided, (long long)left);
}

// The draw is the exact inverse's value or, where the two differ, that of the weights added in value order;
// it is the sums' value whatever the width where U lies at a step
void sums() {
    int64_t differ = 0;
    for (int i = 0; i < 6000; ++i) {
        const uint32_t W = (uint32_t)log_uniform(2.0, i % 10 == 0 ? 3e5 : 3000.0);
        const double beta = log_uniform(1e-3, 1e3);
        const double slope = std::max(1.0, std::rint((i % 2 ? log_uniform(1e-4, 60.0) / W : log_uniform(1e-5, 1000.0)) / beta));
        const bool top = g() % 2;
        const double U = i % 20 == 0 ? 0.0 : u_near_step(slope, beta, W, top);
        const int64_t a = top ? -(int64_t)slope : (int64_t)slope;
        const uint32_t j = (uint32_t)sa::linear_draw(a, 0, W, beta, U);
        const uint32_t by_sums = plain_sums(top, slope, W, beta, U), exact = index_of(exact_x(slope, beta, W, top, U), W);
        if (sa::linear_draw_by_sums(top, slope, W, beta, U) != by_sums) fail("sums without the zero weights", beta * slope, W, top, U);
        if (U == 0.0 ? j != by_sums : j != by_sums && j != exact) fail("draw", beta * slope, W, top, U);
        differ += by_sums != exact;
    }
    std::printf("sums and exact inverse differ in %lld\n", (long long)differ);
    // wider than 65536 values, U at the step itself
    for (int i = 0; i < 40; ++i) {
        const uint32_t W = 65537u + (uint32_t)(g() % 200000);
        const double beta = log_uniform(0.1, 20.0) / W;
        const bool top = g() % 2;
        const double U = u_near_step(1.0, beta, W, top);
        Quad d = exact_x(1.0, beta, W, top, U);
        d = fabsq(d - rintq(d));
        if (d > (Quad)(1e-10 + 1e-14 * W) / 2) continue;
        if ((uint32_t)sa::linear_draw(top ? -1 : 1, 0, W, beta, U) != plain_sums(top, 1.0, W, beta, U))
            fail("wide range at a step", beta, W, top, U);
    }
}

// A margin that freezes a variable in the settled sweeps (the kept bits, as a signed number, at or above
// those of 746 / beta) leaves it where it is for every U, the extremes among them
void margins() {
    int64_t frozen = 0;
    for (int i = 0; i < 400000; ++i) {
        const int64_t lo = -(int64_t)(g() % 50), hi = lo + 1 + (int64_t)(g() % 60);
        const int64_t zk = g() % 2 ? lo : hi, a = (int64_t)(log_uniform(1.0, 1e9)) * (g() % 2 ? 1 : -1);
        const double beta = log_uniform(1e-6, 1e4);
        const bool closed = g() % 2;
        const float t = (float)(746.0 / beta) * 1.000001f;
        uint32_t tb;
        std::memcpy(&tb, &t, 4);
        if ((int16_t)sa::linear_margin(closed, a, lo, hi, zk) < (int16_t)((tb >> 16) + 1u)) continue;
        ++frozen;
        for (double U : {0.0, 0x1p-53, 0.5, 1.0 - 0x1p-52, 1.0 - 0x1p-53}) {
            const uint32_t W = (uint32_t)(hi - lo + 1);
            const int64_t v = closed ? sa::heat_bath_closed(a, lo, W, beta, U, 12345u) : sa::linear_draw(a, lo, W, beta, U);
            if (v != zk) fail(closed ? "frozen, closed form" : "frozen", beta * (double)std::abs(a), W, a < 0, U);
        }
    }
    // after a change of a dense problem: not known, but for the places past the last variable
    for (int32_t n = 1; n <= 70; ++n)
        for (int32_t i = 0; i < n; i += 4) {
            const uint64_t w = sa::cleared_margins(i, n);
            for (int32_t q = 0; q < 4; ++q)
                if ((uint16_t)(w >> (16 * q)) != (i + q < n ? 0 : sa::kFixed)) fail("cleared margins", (double)i, (uint32_t)n, false, q);
        }
    std::printf("frozen %lld\n", (long long)frozen);
    if (frozen < 1000) fail("some freeze", 0, 0, false, 0);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string which = argc > 1 ? argv[1] : "";
    if (which == "single") single();
    else if (which == "decided") decided();
    else if (which == "sums") sums();
    else if (which == "margins") margins();
    else return 2;
    if (failures) {
        std::fprintf(stderr, "%d failures\n", failures);
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
