// sa_settled.h -- the rest of a run once its replicas have settled: one wave per replica sweeps 64
// variables at a time.
//
// Under geometric cooling more than half of a run's sweeps change next to nothing (of the N = 2000
// HUIO problem's sweeps, 60 % change fewer than 1 % of the variables each), and a visit that changes
// nothing costs as much as one that does.  Once a sweep has changed few variables (settled_share),
// the replica comes here, with the coefficients cached in LDS (the paper's caches, Sec. 3.2):
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
// reads 49.4 to 2.25 ms; FC p = 2, u = 100 heat bath, 300 sweeps x 1000 reads 56.4 to 34.3 ms; ML
// p = 10 optimal transition, 300 sweeps x 100 reads 42.5 to 18.9 ms; one-shot HUIO N = 30 heat bath,
// 100 sweeps x 8 reads 2.6 to 1.7 ms.
//
// It is a kernel of its own (a second launch) because inlined into the ordinary kernels it cost their
// sweeps registers: 460 spilled scalars instead of 114 in the wide heat-bath variant, whose ordinary
// sweeps became 1.4 times slower.
//
// A variable whose dE is linear and whose terms hold at most three other factors (SchedRec::pad[1],
// "cached") keeps a_k^(1) modulo 2^32 in ca (its true value fits: DevProblem::coef32); a change of
// another variable adds the change of each shared term's product.  Any other variable keeps in cm
// the smallest energy rise M of a move away from z_k, rounded down to the upper half of a float; 0
// when it is not known, or not positive.  A change of a variable sharing a term sets it to 0.  The
// dense form keeps c1 (int64) for every variable instead.
#pragma once

#include "sa_device.h"

namespace sa {
namespace {

// cm of a linear variable known to have a_k^(1) = 0: every value has the same energy
constexpr uint16_t kFlat = 0x8000;
// e^(-beta M) = 0 in the device's exponential (exp_nonpos clamps there)
constexpr double kSettledArg = 746.0;

// The replica as the sweep's functions take it, with its caches in LDS.
struct SettleView {
    ReplicaCtx R;
    const SchedRec *order;
    int32_t n_order;
    uint32_t *ca;
    uint16_t *cm;
};

__device__ __forceinline__ uint16_t margin_bits(int64_t M) {
    if (M <= 0) return 0;
    // below M after the conversion's rounding, then cut to 16 bits (toward zero)
    const float f = (float)M * 0.9999998f;
    return (uint16_t)(__float_as_uint(f) >> 16);
}
__device__ __forceinline__ double margin_value(uint16_t b) { return (double)__uint_as_float((uint32_t)b << 16); }

// ca of every cached variable from the state, and no margins known: one variable per lane.
template <typename ZT>
__device__ __forceinline__ void settled_init(const SettleView &S, const ZT *z, int lane) {
    const DevProblem &P = S.R.P;
    for (int32_t i = lane; i < S.n_order; i += kWave) {
        const SchedRec sl = S.order[i];
        if (S.cm) S.cm[sl.k] = 0;
        if (S.ca && (sl.pad[1] & 1)) {
            uint32_t acc = 0;
            for (int32_t q = 0; q < sl.deg; ++q) {
                int e;
                acc += record_product<uint32_t, ZT>(P, z, P.inc[sl.row + q], (uint64_t)P.inc_coef[sl.row + q], e);
            }
            S.ca[sl.k] = acc;
        }
    }
}

// After z_k moved from zk to v: the caches of the variables that share a term with k.  Lane l takes
// the row's records l, l + 64, ...
template <typename ZT>
__device__ __forceinline__ void settled_scatter(const SettleView &S, const ZT *z, int32_t k, int32_t row, int32_t deg,
                                                int64_t zk, int64_t v, int lane) {
    const DevProblem &P = S.R.P;
    // (a flat variable's own value does not enter its coefficient: it stays flat)
    if (S.cm && S.cm[k] != kFlat) S.cm[k] = 0;
    for (int32_t c0 = 0; c0 < deg; c0 += kWave) {
        IncRec r;
        uint64_t coef;
        load_record(P, row, deg, c0, lane, r, coef);
        const int e = (int)(r.meta & 0xFFu);
        const int no = (int)(r.meta >> 8);
        if (no > 3) {
            for (int32_t f = 0; f < no; ++f) S.cm[P.overflow[r.o[0] + f]] = 0;
        } else if (no > 0) {
            if (S.ca) {
                const uint32_t g = (uint32_t)coef * (upow<uint32_t>((uint32_t)v, e) - upow<uint32_t>((uint32_t)zk, e));
                const uint32_t z0 = (uint32_t)(int32_t)z[r.o[0]];
                const uint32_t z1 = no > 1 ? (uint32_t)(int32_t)z[r.o[1]] : 1u;
                const uint32_t z2 = no > 2 ? (uint32_t)(int32_t)z[r.o[2]] : 1u;
                atomicAdd(&S.ca[r.o[0]], g * z1 * z2);
                if (no > 1) atomicAdd(&S.ca[r.o[1]], g * z0 * z2);
                if (no > 2) atomicAdd(&S.ca[r.o[2]], g * z0 * z1);
            }
            if (S.cm) {
                S.cm[r.o[0]] = 0;
                if (no > 1) S.cm[r.o[1]] = 0;
                if (no > 2) S.cm[r.o[2]] = 0;
            }
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
                                                   int64_t zk, int lane) {
    const int64_t a1 = to_i64<Acc>(C.a[1]), hi = lo + W - 1;
    if (kE == 1 || (em & ~2u) == 0) return a1 == 0 ? kFlat : margin_bits(zk == lo ? a1 : zk == hi ? -a1 : 0);
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
    if (kRule == SA_HEAT_BATH || kRule == SA_HEAT_BATH_CLOSED) {
        if constexpr (kE == kMaxE) {
            if (kRule == SA_HEAT_BATH_CLOSED && linear)
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
        const uint16_t m = settled_margin(C, em, lo, W, zk, lane);
        if (lane == 0) S.cm[k] = m;
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

// One settled sweep of one replica (one wave).  kDense: the dense form with its coefficient cache
// (c1; the changes keep it exact), else the incidence form with ca and cm.  Adds to H
// the changes of the state hash (tracing) and to `moves` their number; the energy is
// formed from the state at the end of the run.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc, typename ZT>
__device__ __forceinline__ void settled_sweep(const SettleView &S, ZT *z, int lane, int32_t s, double beta, double r_opt,
                                              ScanCarry &cy, uint64_t &H, uint32_t &moves) {
    const ReplicaCtx &R = S.R;
    const DevProblem &P = R.P;
    constexpr bool kEnumerated = kRule == SA_HEAT_BATH;
    constexpr bool kClosed = kRule == SA_HEAT_BATH_CLOSED;
    constexpr bool kHeatBath = kEnumerated || kClosed;
    auto slot = [&](int32_t i) {
        SchedRec m;
        if (i < S.n_order) {
            m = S.order[i];
        } else {
            m.k = -1;
            m.lo = 0;
            m.width = 1;
            m.row = 0;
            m.deg = 0;
            m.emask = 0;
            m.pad[1] = 1;   // (an idle lane reads ca where there is one, as a cached variable does)
        }
        return m;
    };
    SchedRec nx = slot(lane);
    for (int32_t b = 0; b < S.n_order; b += kWave) {
        const SchedRec sl = nx;
        nx = slot(b + kWave + lane);   // loaded under this block's work
        const bool valid = sl.k >= 0;
        const int32_t kk = valid ? sl.k : 0;
        const int64_t lo = sl.lo, hi = lo + (int64_t)(uint32_t)sl.width - 1;
        const uint32_t W32 = (uint32_t)sl.width;
        const int64_t zk = (int64_t)z[kk];
        const bool linear = (sl.emask & ~2u) == 0;
        const bool has_ca = kDense || (S.ca && (sl.pad[1] & 1));
        bool cached = has_ca;   // a1 is known (also of a flat variable without a cached coefficient)
        const int64_t a2 = kDense && valid ? P.d[kk] : 0;
        int64_t a1 = 0;    // cached: a_k^(1)
        double M = 0.0;    // smallest rise of a move away from z_k; <= 0: not known, or there is none
        auto read_caches = [&] {
            if (has_ca) {
                a1 = kDense ? R.c1[kk] : (int64_t)(int32_t)S.ca[kk];
                if (kDense && !linear) M = (double)quadratic_margin(a1, a2, lo, hi, zk);
                else M = zk == lo ? (double)a1 : zk == hi ? -(double)a1 : 0.0;
            } else {
                const uint16_t m = S.cm[kk];
                M = margin_value(m);   // (-0.0 for a flat one)
                cached = m == kFlat;
            }
        };
        read_caches();
        // Settled whatever the random words: every other value's acceptance or weight is exactly 0.
        // (The closed-form draw at the top of the range depends on U = 0, so it reads its words.)
        const bool frozen = beta * M >= kSettledArg && !(kClosed && linear && zk != lo);
        if (__ballot(valid && !frozen) == 0) continue;
        uint32_t x0 = (uint32_t)sl.k, x1 = (uint32_t)s, x2 = R.read, x3 = R.instance_id;
        philox4x32_10(x0, x1, x2, x3, R.key0, R.key1);
        const double U = (double)((((uint64_t)x2 << 32) | x3) >> 11) * 0x1p-53;
        uint64_t todo = ~0ull;
        for (;;) {
            // want: 0 stays, 1 changes to v (energy change d), 2 needs a visit
            int want = 0;
            int64_t v = zk, d = 0;
            if (kHeatBath) {
                if (kClosed && cached && linear) {
                    v = heat_bath_closed(a1, lo, (int64_t)W32, beta, U, x1);
                    d = a1 * (v - zk);
                    want = v != zk ? 1 : 0;
                } else {
                    want = 2;
                    if (M > 0.0) {
                        const double ex = exp_nonpos(-(beta * M));
                        // linear: the values at distance d weigh ex^d on one side; convex: at most
                        // that on either side; else at most ex each
                        const double rho = cached ? (linear ? geometric_tail(ex)
                                                            : a2 >= 0 ? 2.0 * geometric_tail(ex) : (double)(W32 - 1u) * ex)
                                                  : (double)(W32 - 1u) * ex;
                        want = heat_bath_stays(rho, U) ? 0 : 2;
                    }
                }
            } else if (cached && (kRule == SA_METROPOLIS || linear || !((double)x0 * 0x1p-32 < r_opt))) {
                if (kRule == SA_OPT_METROPOLIS && (double)x0 * 0x1p-32 < r_opt) {
                    v = a1 >= 0 ? lo : hi;
                } else {
                    v = lo + (int64_t)(((uint64_t)x1 * (uint64_t)(W32 - 1u)) >> 32);
                    if (v >= zk) v += 1;
                }
                d = kDense ? (v - zk) * (a1 + a2 * (v + zk)) : a1 * (v - zk);
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
                    if (kEnumerated && !kDense && cj) {
                        Coeffs<kMaxE, Acc> C;
#pragma unroll
                        for (int m = 0; m <= kMaxE; ++m) C.a[m] = 0;
                        C.a[1] = (Acc)lane_read64((uint64_t)a1, j);
                        vj = heat_bath_pick<kRegChunk, kMaxE, Acc>(C, loj, Wj, zj, beta, Uj, lane, true, cy);
                        dj = to_i64<Acc>(C.a[1] * (Acc)(vj - zj));
                    } else if constexpr (kDense) {
                        IncRec none;
                        none.meta = 0;
                        none.o[0] = none.o[1] = none.o[2] = 0;
                        taken = update_rule<kRule, kRegChunk, kMaxE, Acc, ZT>(R, z, kj, loj, Wj, em, row, deg, r0, r1, Uj,
                                                                              zj, beta, r_opt, lane, none, 0, P.d[kj], cy,
                                                                              [] {}, vj, dj);
                    } else {
                        taken = settled_visit<kRule, kRegChunk, kMaxE, Acc, ZT>(S, z, kj, loj, Wj, em, row, deg, r0, r1, Uj,
                                                                                zj, beta, r_opt, lane, cy, vj, dj);
                    }
                    changed = taken && vj != zj;
                }
                if (changed) {
                    moves += 1;
                    z[kj] = (ZT)vj;   // every lane stores the same value
                    if (R.trace) H += hash_word(kj, vj) - hash_word(kj, zj);
                    if (kDense) dense_cache_update(P, R.c1, kj, vj - zj, lane, nullptr);
                    else settled_scatter(S, z, kj, row, deg, zj, vj, lane);
                }
                state_write_fence<true>();
            }
            if (!changed) break;
            read_caches();
        }
    }
}

// The settled part of a run: read blockIdx.x from the state in z_out and the sweep in e_out to the end of
// the schedule, or to where it has come unsettled (more than A.leave changes in each of three sweeps
// on end); leaves the state and the next sweep there.
template <bool kDense, int kRule, int kRegChunk, int kMaxE, typename Acc>
__global__ void __launch_bounds__(kWave) settled_kernel(AnnealArgs A) {
    extern __shared__ int32_t lds_state[];
    const int lane = (int)threadIdx.x;
    const int read = (int)blockIdx.x;
    if (read >= A.n_reads) return;
    int32_t s = (int32_t)A.e_out[read];
    if (s >= A.s_end) return;   // uniform
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
    S.n_order = A.n_order;
    R.c1 = kDense ? (int64_t *)((char *)lds_state + A.off_c) : nullptr;
    S.ca = !kDense && A.off_c >= 0 ? (uint32_t *)((char *)lds_state + A.off_c) : nullptr;
    S.cm = !kDense && A.off_m >= 0 ? (uint16_t *)((char *)lds_state + A.off_m) : nullptr;
    state_write_fence<true>();
    if (kDense) dense_cache_init(A.P, z, R.c1, lane, kWave);
    else settled_init(S, z, lane);
    state_write_fence<true>();
    ScanCarry cy;
    int busy = 0;   // sweeps on end past A.leave
    for (; s < A.s_end; ++s) {
        uint64_t H = 0;
        uint32_t moves = 0;
        const double beta = A.beta[s];
        const double r_opt =
            A.otm_r >= 0.0 ? A.otm_r : (A.n_sweeps > 1 ? (double)s / (double)(A.n_sweeps - 1) : 0.0);
        settled_sweep<kDense, kRule, kRegChunk, kMaxE, Acc, int32_t>(S, z, lane, s, beta, r_opt, cy, H, moves);
        if (R.trace && H != 0 && lane == 0) atomicAdd((unsigned long long *)&R.trace[s], (unsigned long long)H);
        busy = moves > (uint32_t)A.leave ? busy + 1 : 0;
        if (busy == 3) {
            ++s;
            break;
        }
    }
    for (int32_t k = lane; k < n; k += kWave) zo[k] = z[k];
    if (lane == 0) A.e_out[read] = s;
}

}  // namespace
}  // namespace sa
