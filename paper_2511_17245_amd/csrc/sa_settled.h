// sa_settled.h -- the rest of a run once its replicas have settled: one wave per replica sweeps 64
// variables at a time.
//
// Under geometric cooling more than half of a run's sweeps change next to nothing (of the N = 2000
// HUIO problem's sweeps, 60 % change fewer than 1 % of the variables each), and a visit that changes
// nothing costs as much as one that does.  Once their sweeps change few variables (settled_share), the
// replicas come here, with the coefficients cached in LDS (the paper's caches, Sec. 3.2):
//  - each lane decides from its variable's cache and random words whether the update changes it:
//    exactly for Metropolis, the closed-form draw and the ends taken by the optimal transition, and
//    from a bound on the other values' weight for the heat bath; lanes that cannot tell ask for a
//    visit.  Where every lane's other values have weight 0 at this temperature (e^(-beta dE) underflows)
//    the random words are not even formed;
//  - the first lane (in index order) that changes or asks is served -- its change applied, or its
//    variable visited by the whole wave as in an ordinary sweep -- and after a change the caches of
//    the variables it shares a term with are brought up to date and the lanes behind it decide again.
// Every lane ahead of the served one has decided "no change" from the same state the index-order
// sweep would show it, so the states, energies and random words are those of the ordinary sweep.
//
// What bounds it: in a settled sweep, the latency of one block's chain (slots, caches, decision: about
// 250 cycles per 64 variables while all are frozen, 700 with their random words); before that, the
// visits.  Measured, ordinary sweeps only against this: dense N = 100 Metropolis, 1000 sweeps x 16
// reads 49.4 to 2.6 ms; FC p = 2, u = 100 heat bath, 300 sweeps x 1000 reads 56.4 to 34.5 ms (18.9 with
// the draws in single precision); ML p = 10 optimal transition, 300 sweeps x 100 reads 42.5 to 18.6 ms; HUIO
// N = 2000, 300 sweeps x 1024 reads 48.0 to 24.9 ms (optimal transition) and 42.6 to 28.6 ms (Metropolis);
// one-shot HUIO N = 30 heat bath, 100 sweeps x 8 reads 2.3 to 1.5 ms.
//
// It is a kernel of its own (a second launch) because inlined into the ordinary kernels it cost their
// sweeps registers: 460 spilled scalars instead of 114 in the wide heat-bath variant, whose ordinary
// sweeps became 1.4 times slower.
//
// A variable whose terms hold it to the first or second power, and in whose terms no variable has more
// than three other factors (SchedRec::pad[1], "cached"), keeps a_k^(1) in ca, and a_k^(2) in cb when some term
// holds a square, modulo 2^32 where every coefficient fits (DevProblem::coef32), else modulo 2^64; a
// change of another variable adds the change of each shared term's product.  The dense form keeps c1 (int64) for every variable.  Every variable
// also has in cm, when it is known, the smallest energy rise M of a move away from z_k, rounded down to
// the upper half of a float; 0 when it is not known, or not positive; with the sign set where it may not
// freeze the variable (linear_margin); kFlat and kFixed for variables whose values all have the same energy and
// that are fixed (sa_draw.h).  A change of a variable sharing a
// term sets it to 0, the next decision of a cached variable and the next visit of another finds it
// again.  A sweep first reads cm alone, four variables per lane, and skips the blocks of 64 whose
// variables are all frozen: beta M >= 746, where every other value's acceptance or weight is exactly 0.
#pragma once

#include "sa_device.h"

namespace sa {
namespace {

template <int k>
struct Int {
    static constexpr int value = k;
};
// e^(-beta M) = 0 in the device's exponential (exp_nonpos clamps there)
constexpr double kSettledArg = 746.0;

// The replica as the sweep's functions take it, with its caches in LDS.
struct SettleView {
    ReplicaCtx R;
    const SchedRec *order;   // every variable in index order (k = -1 for a fixed one)
    bool closed;         // heat bath: the closed-form draw where dE is linear
    bool small;          // cached coefficients fit 32 bits, and every value 30
    bool wide;           // ca and cb hold 64-bit words
    void *ca, *cb;       // nullptr where no variable is cached / none has a square
    uint16_t *cm;        // whole groups of four
};

// (without the sign: 0 for a flat variable)
__device__ __forceinline__ double margin_value(uint16_t b) { return (double)__uint_as_float((uint32_t)(b & 0x7FFFu) << 16); }

// a cached coefficient of variable i
__device__ __forceinline__ int64_t cache_read(const SettleView &S, const void *c, int32_t i) {
    return S.wide ? ((const int64_t *)c)[i] : (int64_t)((const int32_t *)c)[i];
}

// The coefficients of every cached variable from the state, and no margins known: one variable per lane.
// (Products and sums modulo 2^64; the low words are those modulo 2^32.)
template <typename ZT>
__device__ __forceinline__ void settled_init(const SettleView &S, const ZT *z, int lane) {
    const DevProblem &P = S.R.P;
    for (int32_t i = lane; i < ((P.n + 3) & ~3); i += kWave) {
        SchedRec sl;
        sl.k = -1;
        if (i < P.n) sl = S.order[i];
        S.cm[i] = sl.k >= 0 ? 0 : kFixed;
        if (sl.k >= 0 && S.ca && sl.pad[1]) {
            uint64_t a1 = 0, a2 = 0;
            for (int32_t q = 0; q < sl.deg; ++q) {
                int e;
                const uint64_t p =
                    record_product<uint64_t, ZT>(P, z, P.inc[sl.row + q], (uint64_t)P.inc_coef[sl.row + q], e);
                a1 += e == 1 ? p : 0u;
                a2 += e == 2 ? p : 0u;
            }
            if (S.wide) ((uint64_t *)S.ca)[i] = a1;
            else ((uint32_t *)S.ca)[i] = (uint32_t)a1;
            if (S.cb) {
                if (S.wide) ((uint64_t *)S.cb)[i] = a2;
                else ((uint32_t *)S.cb)[i] = (uint32_t)a2;
            }
        }
    }
}

// One record's other factors i0, i1, i2 (sorted; -1 where there are fewer): z_k^e moved from zk^e to v^e.
// A factor that occurs once moves its variable's a^(1), one that occurs twice its a^(2) (three times:
// not a cached variable).
template <typename Part, typename Word, typename ZT>
__device__ __forceinline__ void scatter_record(Word *ca, Word *cb, const ZT *z, uint64_t coef, int e, int64_t zk, int64_t v,
                                               int32_t i0, int32_t i1, int32_t i2) {
    const Part g = (Part)coef * (upow<Part>((Part)v, e) - upow<Part>((Part)zk, e));
    const Part z0 = (Part)(int64_t)z[i0];
    const Part z1 = i1 >= 0 ? (Part)(int64_t)z[i1] : (Part)1;
    const Part z2 = i2 >= 0 ? (Part)(int64_t)z[i2] : (Part)1;
    if (i0 != i1) {
        atomicAdd(&ca[i0], (Word)(g * z1 * z2));
        if (i1 >= 0 && i1 != i2) {
            atomicAdd(&ca[i1], (Word)(g * z0 * z2));
            if (i2 >= 0) atomicAdd(&ca[i2], (Word)(g * z0 * z1));
        } else if (i2 >= 0 && cb) {
            atomicAdd(&cb[i1], (Word)(g * z0));
        }
    } else if (i1 != i2) {
        if (cb) atomicAdd(&cb[i0], (Word)(g * z2));
        if (i2 >= 0) atomicAdd(&ca[i2], (Word)(g * z0 * z1));
    }
}

// After z_k moved from zk to v: the caches of the variables that share a term with k.  Lane l takes
// the row's records l, l + 64, ...
template <typename ZT>
__device__ __forceinline__ void settled_scatter(const SettleView &S, const ZT *z, int32_t k, int32_t row, int32_t deg,
                                                int64_t zk, int64_t v, int lane) {
    const DevProblem &P = S.R.P;
    // (a flat variable's own value does not enter its coefficient: it stays flat)
    if (S.cm[k] != kFlat) S.cm[k] = 0;
    for (int32_t c0 = 0; c0 < deg; c0 += kWave) {
        IncRec r;
        uint64_t coef;
        load_record(P, row, deg, c0, lane, r, coef);
        const int e = (int)(r.meta & 0xFFu);
        const int no = (int)(r.meta >> 8);
        if (no > 3) {
            for (int32_t f = 0; f < no; ++f) S.cm[P.overflow[r.o[0] + f]] = 0;
        } else if (no > 0) {
            const int32_t i0 = r.o[0], i1 = no > 1 ? r.o[1] : -1, i2 = no > 2 ? r.o[2] : -1;
            if (S.ca) {
                if (S.wide) scatter_record<uint64_t>((unsigned long long *)S.ca, (unsigned long long *)S.cb, z, coef, e, zk, v, i0, i1, i2);
                else scatter_record<uint32_t>((uint32_t *)S.ca, (uint32_t *)S.cb, z, coef, e, zk, v, i0, i1, i2);
            }
            S.cm[i0] = 0;
            if (no > 1) S.cm[i1] = 0;
            if (no > 2) S.cm[i2] = 0;
        }
    }
}

// The smallest dE(v), v != z_k, of a polynomial of degree at most two: on either side of z_k it lies
// next to z_k or at the range's end (a concave dE's minimum over a range is at an end of it, a convex
// one that rises on both sides of z_k keeps rising, and one that does not gives a value <= 0 here).
__device__ __forceinline__ int64_t quadratic_margin(int64_t a1, int64_t a2, int64_t lo, int64_t hi, int64_t zk) {
    auto de = [&](int64_t v) { return (v - zk) * (a1 + a2 * (v + zk)); };
    int64_t M = INT64_MAX;
    if (zk < hi) {
        const int64_t p = de(zk + 1), q = de(hi);
        M = p < q ? p : q;
    }
    if (zk > lo) {
        const int64_t p = de(zk - 1), q = de(lo);
        M = p < M ? p : M;
        M = q < M ? q : M;
    }
    return M;
}

// Margin of a variable that a visit left at z_k, from its coefficients (wave-uniform).
template <int kE, typename Acc>
__device__ __forceinline__ uint16_t settled_margin(const Coeffs<kE, Acc> &C, uint32_t em, int64_t lo, int64_t W,
                                                   int64_t zk, bool closed, int lane) {
    const int64_t a1 = to_i64<Acc>(C.a[1]), hi = lo + W - 1;
    if (kE == 1 || (em & ~2u) == 0) return linear_margin(closed, a1, lo, hi, zk);
    if (kE == 2 || (em & ~6u) == 0)
        return margin_bits(quadratic_margin(a1, to_i64<Acc>(C.a[kE >= 2 ? 2 : 1]), lo, hi, zk));
    if (W > 16 * kWave) return 0;   // not worth the enumeration
    int64_t M = INT64_MAX;
    for (int64_t i = lane; i < W; i += kWave) {
        const int64_t d = poly_delta(C, zk, lo + i);
        M = lo + i != zk && d < M ? d : M;
    }
    return margin_bits(wave_min_i64(M));
}

// A settled sweep's visit of a variable without a cached coefficient: update_rule, with the
// coefficients formed once for the rule and, when nothing changes, for the margin.
template <int kRule, int kRegChunk, int kMaxE, typename Acc, typename ZT>
__device__ __forceinline__ bool settled_visit(const SettleView &S, const ZT *z, int32_t k, int64_t lo, int64_t W, uint32_t em,
                                              int32_t row, int32_t deg, uint32_t r0, uint32_t r1, double U, int64_t zk,
                                              double beta, double r_opt, int lane, ScanCarry &cy, int64_t &v, int64_t &d) {
    const DevProblem &P = S.R.P;
    // the Metropolis kernels take any exponent (kMaxE = 1 there); one above four gets no margin
    constexpr int kE = kRule == SA_METROPOLIS ? 4 : kMaxE;
    IncRec rec;
    uint64_t rc;
    load_record(P, row, deg, 0, lane, rec, rc);
    if (kRule == SA_METROPOLIS && (em >> (kE + 1)) != 0)
        return update_rule<kRule, kRegChunk, kMaxE, Acc, ZT>(S.R, z, k, lo, W, em, row, deg, r0, r1, U, zk, beta, r_opt, lane,
                                                             rec, rc, 0, cy, [] {}, v, d);
    Coeffs<kE, Acc> C;
    row_coeffs<kE, Acc, ZT>(P, z, k, row, deg, em, lane, rec, rc, C);
    const bool linear = kE == 1 || (em & ~2u) == 0;
    bool taken = true;
    if (kRule == SA_HEAT_BATH) {
        if constexpr (kE == kMaxE) {
            if (S.closed && linear)
                v = heat_bath_closed(to_i64<Acc>(C.a[1]), lo, W, beta, U, r1);
            else
                v = heat_bath_pick<kRegChunk, kMaxE, Acc>(C, lo, W, zk, beta, U, lane, linear, cy);
            d = poly_delta(C, zk, v);
        }
    } else {
        if (kRule == SA_OPT_METROPOLIS && (double)r0 * 0x1p-32 < r_opt) {
            if (linear) {
                v = to_i64<Acc>(C.a[1]) >= 0 ? lo : lo + W - 1;
                d = to_i64<Acc>(C.a[1] * (Acc)(v - zk));
            } else if (kRegChunk == 1 && W > S.R.otm_enum_max && W > kWave) {
                v = argmin_wide<kE, Acc>(C, lo, W, zk, lane, d);
            } else {
                v = argmin_range<kE, Acc>(C, lo, W, zk, lane, d);
            }
        } else {
            v = lo + (int64_t)(((uint64_t)r1 * (uint64_t)(W - 1)) >> 32);
            if (v >= zk) v += 1;
            d = poly_delta(C, zk, v);
        }
        taken = metropolis_accept(d, beta, U);
    }
    if (!taken || v == zk) {
        const uint16_t m = settled_margin(C, em, lo, W, zk, kRule == SA_HEAT_BATH && S.closed, lane);
        if (lane == 0) S.cm[k] = m;   // (k: its place in index order)
    }
    return taken;
}

// Whether a heat-bath draw stays at z_k for certain: the other values' weights sum to at most rho
// (weights relative to z_k's, the largest), so every cumulative weight below z_k's is at most rho, the
// total at most 1 + rho, and U lies well inside (rho, 1 / (1 + rho)).  The slack of 1e-9 and 1e-12 is
// far above the rounding of any summation order.
__device__ __forceinline__ bool heat_bath_stays(double rho, double U) {
    rho *= 1.0 + 1e-9;
    return U > rho && U * (1.0 + rho) < 1.0 - 1e-12;
}
// sum over d >= 1 of e^(-c d), from e1 = e^(-c); no bound above e1 = 1/2
__device__ __forceinline__ double geometric_tail(double e1) { return e1 < 0.5 ? e1 / (1.0 - e1) : 1e300; }

// Optimal transition of a variable with exponents one and two (quad_argmin_quadratic's candidates, all
// in one lane): the value of smallest dE over the range, z_k included, ties to the lowest.
__device__ __forceinline__ int64_t lane_argmin_quadratic(int64_t a1, int64_t a2, int64_t lo, int64_t hi, int64_t zk) {
    int64_t f = lo;
    if (a2 > 0) {
        const double t = -(double)a1 / (2.0 * (double)a2);
        f = t < (double)lo ? lo : t > (double)hi ? hi : (int64_t)__builtin_floor(t);
    }
    int64_t best = INT64_MAX, bv = INT64_MAX;
    for (int i = 0; i < 7; ++i) {
        int64_t v = i == 0 ? lo : i == 1 ? hi : i == 2 ? zk : f + (int64_t)(i - 4);
        v = v < lo ? lo : v > hi ? hi : v;
        const int64_t d = (v - zk) * (a1 + a2 * (v + zk));
        if (d < best || (d == best && v < bv)) {
            best = d;
            bv = v;
        }
    }
    return bv;
}

// One block of 64 variables (slots sl, one per lane) of a settled sweep.  Returns the number of changes.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc, typename ZT>
__device__ __forceinline__ uint32_t settled_block(const SettleView &S, ZT *z, int lane, int32_t b, const SchedRec &sl,
                                                  int32_t s, double beta, double r_opt, int16_t thr, ScanCarry &cy,
                                                  uint64_t &H, int64_t &E) {
    const ReplicaCtx &R = S.R;
    const DevProblem &P = R.P;
    constexpr bool kHeatBath = kRule == SA_HEAT_BATH;
    const bool closed = kHeatBath && S.closed;
    uint32_t moves = 0;
    const bool valid = sl.k >= 0;
    const int32_t kk = valid ? sl.k : 0;
    const int64_t lo = sl.lo, hi = lo + (int64_t)(uint32_t)sl.width - 1;
    const uint32_t W32 = (uint32_t)sl.width;
    const int64_t zk = (int64_t)z[kk];
    const bool linear = (sl.emask & ~2u) == 0;
    const bool has = kDense || (S.ca && sl.pad[1]);
    bool cached = has;         // a1 and a2 are known (also of a flat variable without cached ones)
    int64_t a1 = 0, a2 = 0;
    double M = 0.0;            // smallest rise of a move away from z_k; <= 0: not known, or there is none
    uint16_t mbits = 0;        // as cm keeps it
    if (kDense && valid) a2 = P.d[kk];
    // no variable of the block has a square; dE from 32-bit factors where coefficients and values allow
    const bool all_linear = __ballot(valid && !linear) == 0;
    auto de = [&](int64_t v) -> int64_t {
        if (S.small) {
            const int32_t dv = (int32_t)v - (int32_t)zk, sv = (int32_t)v + (int32_t)zk;
            if (all_linear) return (int64_t)(int32_t)a1 * (int64_t)dv;
            return ((int64_t)(int32_t)a1 + (int64_t)(int32_t)a2 * (int64_t)sv) * (int64_t)dv;
        }
        return (v - zk) * (a1 + a2 * (v + zk));
    };
    // The smallest dE(v), v != z_k, of a polynomial of degree at most two: on either side of z_k it lies
    // next to z_k or at the range's end (a concave dE's minimum over a range is at an end of it, a
    // convex one that rises on both sides of z_k keeps rising, and one that does not gives a value <= 0).
    auto find_margin = [&] {
        int64_t m = zk == lo ? a1 : zk == hi ? -a1 : 0;
        if (!all_linear && !linear) {
            m = INT64_MAX;
            if (zk < hi) {
                const int64_t p = de(zk + 1), q = de(hi);
                m = p < q ? p : q;
            }
            if (zk > lo) {
                const int64_t p = de(zk - 1), q = de(lo);
                m = p < m ? p : m;
                m = q < m ? q : m;
            }
        }
        M = (double)m;
        mbits = linear && !may_freeze(closed, lo, zk) ? 0 : margin_bits(m);
    };
    // decisions that read M find it each time; the others only now and then, for cm (below)
    constexpr bool kUsesMargin = kRule != SA_METROPOLIS;
    auto read_caches = [&] {
        if (has) {
            a1 = kDense ? R.c1[kk] : cache_read(S, S.ca, kk);
            if (!kDense && !linear) a2 = cache_read(S, S.cb, kk);
            if (kUsesMargin) find_margin();
        } else {
            mbits = S.cm[kk];
            M = margin_value(mbits);
            cached = mbits == kFlat;
        }
    };
    read_caches();
    auto keep_margins = [&] {
        if (valid ? has : b + lane < P.n) S.cm[b + lane] = !valid ? kFixed : (int64_t)z[kk] == zk ? mbits : 0;
        state_write_fence<true>();
    };
    // Margins that a neighbour's change cleared and that hold all the same: nothing can change here.  (In a warm
    // settled sweep most blocks are of this kind; HUIO of 2000 variables, optimal transition, 1024 reads x 300
    // sweeps: 25.4 -> 24.9 ms.  Metropolis would have to find the margins for it each time: 28.7 -> 31.1 ms.)
    if (kUsesMargin && __ballot(valid && (int16_t)mbits < thr) == 0) {
        keep_margins();
        return 0;
    }
    uint32_t x0 = (uint32_t)sl.k, x1 = (uint32_t)s, x2 = R.read, x3 = R.instance_id;
    philox4x32_10(x0, x1, x2, x3, R.key0, R.key1);
    const double U = (double)((((uint64_t)x2 << 32) | x3) >> 11) * 0x1p-53;
    const bool optimal = kRule == SA_OPT_METROPOLIS && (double)x0 * 0x1p-32 < r_opt;
    uint64_t todo = ~0ull;
    for (;;) {
        // want: 0 stays, 1 changes to v (energy change d), 2 needs a visit
        int want = 0;
        int64_t v = zk, d = 0;
        if (kHeatBath) {
            if (closed && cached && linear) {
                v = heat_bath_closed(a1, lo, (int64_t)W32, beta, U, x1);
                d = a1 * (v - zk);
                want = v != zk ? 1 : 0;
            } else {
                want = 2;
                if (M > 0.0) {
                    const double ex = exp_nonpos(-(beta * M));
                    // linear: the values at distance d weigh ex^d on one side; convex: at most that on
                    // either side; else at most ex each
                    const double rho = !cached || (!linear && a2 < 0) ? (double)(W32 - 1u) * ex
                                       : linear                        ? geometric_tail(ex)
                                                                       : 2.0 * geometric_tail(ex);
                    want = heat_bath_stays(rho, U) ? 0 : 2;
                }
            }
        } else if (cached) {
            if (optimal) {
                v = linear ? (a1 >= 0 ? lo : hi) : M > 0.0 ? zk : lane_argmin_quadratic(a1, a2, lo, hi, zk);
            } else {
                v = lo + (int64_t)(((uint64_t)x1 * (uint64_t)(W32 - 1u)) >> 32);
                if (v >= zk) v += 1;
            }
            d = de(v);
            want = v != zk && metropolis_accept(d, beta, U) ? 1 : 0;
        } else {
            // a positive margin: z_k is the optimal value, and a proposal's rise is at least M
            want = M > 0.0 && U > exp_nonpos(-(beta * M)) * (1.0 + 1e-9) ? 0 : 2;
        }
        uint64_t mask = __ballot(valid && want != 0) & todo;
        bool changed = false;
        while (mask != 0 && !changed) {   // uniform
            const int j = __ffsll((unsigned long long)mask) - 1;
            todo = j == kWave - 1 ? 0ull : ~0ull << (j + 1);
            mask &= todo;
            const int32_t kj = (int32_t)lane_read32((uint32_t)sl.k, j);
            const int32_t row = (int32_t)lane_read32((uint32_t)sl.row, j);
            const int32_t deg = (int32_t)lane_read32((uint32_t)sl.deg, j);
            const int64_t zj = (int64_t)(int32_t)lane_read32((uint32_t)(int32_t)zk, j);
            int64_t vj, dj;
            if (lane_read32((uint32_t)want, j) == 1u) {
                vj = (int64_t)(int32_t)lane_read32((uint32_t)(int32_t)v, j);
                dj = (int64_t)lane_read64((uint64_t)d, j);
                changed = true;
            } else {
                const int64_t loj = (int32_t)lane_read32((uint32_t)sl.lo, j);
                const int64_t Wj = (int64_t)lane_read32((uint32_t)sl.width, j);
                const uint32_t em = lane_read32(sl.emask, j);
                const uint32_t r0 = lane_read32(x0, j), r1 = lane_read32(x1, j);
                const double Uj = __longlong_as_double((long long)lane_read64((uint64_t)__double_as_longlong(U), j));
                const bool cj = kDense || lane_read32(cached ? 1u : 0u, j) != 0;
                bool taken = true;
                if (kHeatBath && cj) {   // an enumerated draw from the cached coefficients
                    Coeffs<kMaxE, Acc> C;
#pragma unroll
                    for (int m = 0; m <= kMaxE; ++m) C.a[m] = 0;
                    C.a[1] = (Acc)lane_read64((uint64_t)a1, j);
                    if (kMaxE >= 2) C.a[kMaxE >= 2 ? 2 : 1] = (Acc)lane_read64((uint64_t)a2, j);
                    vj = heat_bath_pick<kRegChunk, kMaxE, Acc>(C, loj, Wj, zj, beta, Uj, lane, (em & ~2u) == 0, cy);
                    dj = poly_delta(C, zj, vj);
                } else if constexpr (!kDense) {
                    taken = settled_visit<kRule, kRegChunk, kMaxE, Acc, ZT>(S, z, kj, loj, Wj, em, row, deg, r0, r1, Uj, zj,
                                                                            beta, r_opt, lane, cy, vj, dj);
                } else {
                    vj = zj;   // (not reached: the dense form's other rules decide in the lane)
                    dj = 0;
                }
                changed = taken && vj != zj;
            }
            if (changed) {
                moves += 1;
                z[kj] = (ZT)vj;   // every lane stores the same value
                E += dj;
                if (R.trace) H += hash_word(kj, vj) - hash_word(kj, zj);
                if (kDense) {
                    dense_cache_update(P, R.c1, kj, vj - zj, lane, nullptr);
                    for (int32_t i = 4 * lane; i < P.n; i += 4 * kWave) *(uint64_t *)&S.cm[i] = cleared_margins(i, P.n);
                } else {
                    settled_scatter(S, z, kj, row, deg, zj, vj, lane);
                }
            }
            state_write_fence<true>();
        }
        if (!changed) break;
        read_caches();
    }
    // the margins found; a variable that changed here (its z_k no longer the lane's) has none.  (Where no
    // decision reads them they are found every fourth sweep.)
    if (kUsesMargin || (s & 3) == 0) {
        if (!kUsesMargin && has) find_margin();
        keep_margins();
    }
    return moves;
}

// One settled sweep of one replica (one wave).  kDense: the dense form with its coefficient cache
// (c1; the changes keep it exact), else the incidence form.  Adds to H the changes of the state hash
// (tracing) and to E those of the energy.  Returns the number of changes.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc, typename ZT>
__device__ __forceinline__ uint32_t settled_sweep(const SettleView &S, ZT *z, int lane, int32_t s, double beta, double r_opt,
                                                  ScanCarry &cy, uint64_t &H, int64_t &E) {
    const int32_t n = S.R.P.n;
    // the least margin bits with beta M >= 746: above 746 / beta rounded up
    const float t = (float)(kSettledArg / beta) * 1.000001f;
    const uint32_t tb = (__float_as_uint(t) >> 16) + 1u;
    const int16_t thr = (int16_t)(tb < (uint32_t)kFixed ? tb : (uint32_t)kFixed);
    auto load = [&](int32_t b) {
        SchedRec m;
        if (b + lane < n) {
            m = S.order[b + lane];
        } else {
            m.k = -1;
            m.lo = 0;
            m.width = 1;
            m.row = 0;
            m.deg = 0;
            m.emask = 0;
            m.pad[1] = 1;
        }
        return m;
    };
    uint32_t moves = 0;
    for (int32_t base = 0; base < n; base += 4 * kWave) {
        // lane l: variables base + 4 l .. + 3; block q of 64 is lanes 16 q .. 16 q + 15
        auto active = [&]() -> uint64_t {
            bool any = false;
            if (base + 4 * lane < n) {
                const uint64_t m = *(const uint64_t *)&S.cm[base + 4 * lane];
                any = (int16_t)m < thr || (int16_t)(m >> 16) < thr || (int16_t)(m >> 32) < thr || (int16_t)(m >> 48) < thr;
            }
            return __ballot(any);
        };
        uint64_t am = active();
        int q = 0;
        auto next = [&](int from) {   // the first block from `from` on with an active variable, or 4
            while (from < 4 && ((am >> (16 * from)) & 0xFFFFull) == 0) ++from;
            return from;
        };
        q = next(0);
        SchedRec sl;
        if (q < 4) sl = load(base + kWave * q);
        while (q < 4) {   // uniform
            int qn = next(q + 1);
            SchedRec sn = sl;
            if (qn < 4) sn = load(base + kWave * qn);   // under this block's work
            const uint32_t c = settled_block<kDense, kRule, kRegChunk, kMaxE, Acc, ZT>(S, z, lane, base + kWave * q, sl, s, beta,
                                                                                       r_opt, thr, cy, H, E);
            moves += c;
            if (c != 0) {
                am = active();
                const int qc = next(q + 1);
                if (qc != qn && qc < 4) sn = load(base + kWave * qc);
                qn = qc;
            }
            sl = sn;
            q = qn;
        }
    }
    return moves;
}

// The settled part of a run of one replica from sweep s: to s_end, or to where it has come unsettled
// (more than twice `limit` changes in each of three stretches of `every` sweeps on end).  `z`: its state in LDS,
// `off_*` the byte offsets of the caches after it.  Returns the next sweep; adds to E the energy changes.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc>
__device__ __forceinline__ int32_t settled_run(SettleView &S, int32_t *z, int lane, int32_t s, int32_t s_end, int32_t off_c,
                                               int32_t off_c2, int32_t off_m, int32_t every, uint32_t limit, int64_t &E) {
    ReplicaCtx &R = S.R;
    R.c1 = kDense ? (int64_t *)((char *)z + off_c) : nullptr;
    S.wide = !R.P.coef32;
    S.ca = !kDense && off_c >= 0 ? (void *)((char *)z + off_c) : nullptr;
    S.cb = !kDense && off_c2 >= 0 ? (void *)((char *)z + off_c2) : nullptr;
    S.cm = (uint16_t *)((char *)z + off_m);
    state_write_fence<true>();
    settled_init(S, z, lane);
    if (kDense) dense_cache_init(R.P, z, R.c1, lane, kWave);
    state_write_fence<true>();
    ScanCarry cy;
    int busy = 0;   // stretches on end past twice `limit`
    uint32_t moves = 0;
    int32_t left = every;
    for (; s < s_end; ++s) {
        uint64_t H = 0;
        const double beta = R.beta[s];
        const double r_opt =
            R.otm_r >= 0.0 ? R.otm_r : (R.n_sweeps > 1 ? (double)s / (double)(R.n_sweeps - 1) : 0.0);
        moves += settled_sweep<kDense, kRule, kRegChunk, kMaxE, Acc, int32_t>(S, z, lane, s, beta, r_opt, cy, H, E);
        if (R.trace && H != 0 && lane == 0) atomicAdd((unsigned long long *)&R.trace[s], (unsigned long long)H);
        if (--left == 0) {
            busy = moves > 2u * limit ? busy + 1 : 0;
            if (busy == 3) return s + 1;
            moves = 0;
            left = every;
        }
    }
    return s;
}

// Plain runs: read blockIdx.x, if it was handed over, from the state in z_out and the sweep in e_out; leaves
// the state and the next sweep there.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc>
__global__ void __launch_bounds__(kWave) settled_kernel(AnnealArgs A) {
    extern __shared__ int32_t lds_state[];
    const int lane = (int)threadIdx.x;
    const int read = (int)blockIdx.x;
    if (read >= A.n_reads) return;
    const int64_t at = (int64_t)lane_read64((uint64_t)A.e_out[read], 0);   // (in scalar registers)
    if (!handed_over(at)) return;   // uniform
    int32_t s = handed_sweep(at);
    const int32_t n = A.P.n;
    int32_t *z = lds_state;
    int32_t *zo = A.z_out + (size_t)read * n;
    for (int32_t k = lane; k < n; k += kWave) z[k] = zo[k];
    SettleView S;
    ReplicaCtx &R = S.R;
    R.P = A.P;
    R.beta = A.beta;
    R.n_sweeps = A.n_sweeps;
    R.key0 = A.key0;
    R.key1 = A.key1;
    R.instance_id = A.instance_id;
    R.read = (uint32_t)read;
    R.otm_r = A.otm_r;
    R.otm_enum_max = A.otm_enum_max;
    R.trace = A.trace ? A.trace + (size_t)read * (size_t)(A.s_end - A.s_begin) - A.s_begin : nullptr;
    S.order = A.order;
    S.small = A.P.coef32 && A.z30;
    S.closed = A.closed != 0;
    int64_t E = 0;   // (the last launch sums the energy of every state)
    s = settled_run<kDense, kRule, kRegChunk, kMaxE, Acc>(S, z, lane, s, A.s_end, A.off_c, A.off_c2, A.off_m,
                                                          A.every, (uint32_t)A.limit, E);
    for (int32_t k = lane; k < n; k += kWave) zo[k] = z[k];
    if (lane == 0) A.e_out[read] = hand_over(s);
}

// Batches and server chunks: task blockIdx.x, a read whose D.next says it has settled.  Leaves its
// state, energy and next sweep (as ~s_end while it stays settled, for the next chunk).
template <int kMaxE>
__global__ void __launch_bounds__(kWave) settled_batch_kernel(const BatchInst *insts, const BatchTask *tasks) {
    extern __shared__ int32_t lds_state[];
    using Acc = uint64_t;
    constexpr int kOtmE = kMaxE < 4 ? kMaxE : 4;
    const int lane = (int)threadIdx.x;
    const BatchTask task = tasks[blockIdx.x];
    const BatchInst &D = insts[task.inst];
    const int32_t read = task.read;
    int32_t s = uni_load(&D.next[read]);
    if (s >= 0 || ~s >= D.s_end) return;   // uniform: not settled, or done
    s = ~s;
    SettleView S;
    ReplicaCtx &R = S.R;
    R.P = D.P;
    const int32_t n = R.P.n;
    int32_t *z = lds_state;
    int32_t *zo = D.z_out + (size_t)read * n;
    for (int32_t k = lane; k < n; k += kWave) z[k] = zo[k];
    R.beta = D.beta;
    R.n_sweeps = D.n_sweeps;
    R.key0 = D.key0;
    R.key1 = D.key1;
    R.instance_id = D.instance_id;
    R.read = (uint32_t)read;
    R.otm_r = -1.0;
    R.otm_enum_max = kOtmEnumMax;
    R.trace = nullptr;
    S.order = D.order;
    S.small = R.P.coef32 && D.z30;
    S.closed = D.rule == SA_HEAT_BATH_CLOSED;
    int64_t E = 0;
    auto go = [&](auto dense, auto rule, auto maxe) {
        s = settled_run<decltype(dense)::value, decltype(rule)::value, 0, decltype(maxe)::value, Acc>(
            S, z, lane, s, D.s_end, D.off_c, D.off_c2, D.off_m, D.every, (uint32_t)D.limit, E);
    };
    auto by_rule = [&](auto dense, auto maxe, auto otm_e) {
        if (D.rule == SA_METROPOLIS) {
            go(dense, Int<SA_METROPOLIS>(), Int<1>());
        } else if (D.rule == SA_OPT_METROPOLIS) {
            go(dense, Int<SA_OPT_METROPOLIS>(), otm_e);
        } else {
            go(dense, Int<SA_HEAT_BATH>(), maxe);
        }
    };
    if (R.P.dense) by_rule(Int<1>(), Int<2>(), Int<2>());
    else by_rule(Int<0>(), Int<kMaxE>(), Int<kOtmE>());
    for (int32_t k = lane; k < n; k += kWave) zo[k] = z[k];
    if (lane == 0) {
        D.e_out[read] += E;
        D.next[read] = s < D.s_end ? s : ~s;
    }
}

}  // namespace
}  // namespace sa
