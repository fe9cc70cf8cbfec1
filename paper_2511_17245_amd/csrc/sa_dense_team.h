// sa_dense_team.h -- dense problems annealed by a team of waves per replica around the coefficient
// cache c1 (Sec. 3.2).
//
// One wavefront per replica spends a dense update on its row: N / 64 products per lane for c1_k, or N / 64
// cached sums per lane after each change, and for the heat bath W / 64 weights per lane; with 16 reads
// of an N = 4096, W = 2001 problem that is 5.7 us per update on 16 of the 1024 SIMDs.  Here the waves
// of a workgroup share one replica: its state and c1 are in LDS, thread t keeps columns 4 t .. 4 t + 3 (of
// each 4 nthr) of c1 up to date, and the heat bath's weights are split over all threads.
//
// Every wave decides every update for itself from the same LDS words (64 variables at a time, one per
// lane, as the settled kernel does), so a sweep needs barriers only where something changes: one after
// a change's cache update and one before it, or for an enumerated heat-bath draw two (the waves' weight
// sums, the drawn value).  While most draws change their variable the lanes' decisions are skipped and every
// variable is drawn at once.  The next variable's coupling row is loaded under the current draw.
//
// What bounds it: the chain of one draw (LDS reads, minimum, exponentials, scan, three barriers): 50 %
// of the wave time waits, 330 VALU instructions per wave and hot draw.  Measured: dense N = 4096,
// W = 2001 heat bath, 20 sweeps x 16 reads 467 to 100 ms (109 before the draws in single precision; hot sweeps
// 33 to 9.5 ms, settled ones 12 to 0.4 ms); a served burst of 18 HUIO and two dense N = 2048 requests 321 to
// 108 ms.
#pragma once

#include "sa_settled.h"

namespace sa {
namespace {

// LDS words the waves exchange: their weight sums and the drawn value, each twice (a draw writes the
// pair the one before it did not, so that no barrier is needed between its writes and earlier reads).
struct TeamExchange {
    double sum[2][16];
    int32_t drawn[2];
};
static_assert(sizeof(TeamExchange) <= kTeamExchangeBytes, "the exchange fits its place");

struct TeamCtx {
    DevProblem P;
    const double *beta;
    int32_t n_sweeps, s_begin, s_end;
    uint32_t key0, key1, instance_id, read;
    double otm_r;
    const SchedRec *order;
    bool closed;
    bool exact53;   // energy differences below 2^52: exact in double
    int tid, nthr;
    uint64_t *trace;   // indexed by the sweep, or nullptr
};

__device__ __forceinline__ double lane_double(double x, int l) {
    return __longlong_as_double((long long)lane_read64((uint64_t)__double_as_longlong(x), l));
}

// c1_i += J_ki dz for this thread's columns; first: its couplings of the first 8 nthr columns (int8
// rows: columns 4 t .. and 4 (nthr + t) ..), loaded ahead.
template <typename C>
__device__ __forceinline__ void team_update(const DevProblem &P, C *c1, int32_t k, int64_t dz, int tid, int nthr,
                                            uint2 first) {
    for (int32_t j0 = 4 * tid; j0 < P.n; j0 += 4 * nthr) {
        int32_t J[4];
        if (P.jbytes == 1) {
            const uint32_t w = j0 == 4 * tid            ? first.x
                               : j0 == 4 * (tid + nthr) ? first.y
                                                        : *(const uint32_t *)((const int8_t *)P.jd +
                                                                              (size_t)k * P.row_stride + j0);
#pragma unroll
            for (int u = 0; u < 4; ++u) J[u] = (int32_t)(int8_t)(w >> (8 * u));
        } else {
            const int4 w = *(const int4 *)((const int32_t *)P.jd + (size_t)k * P.row_stride + j0);
            J[0] = w.x;
            J[1] = w.y;
            J[2] = w.z;
            J[3] = w.w;
        }
        // (c1 is padded to the row stride, its couplings there are zero)
        if constexpr (sizeof(C) == 4) {
            int4 q = *(int4 *)&c1[j0];
            const int32_t dz32 = (int32_t)dz;
            if (P.jbytes == 1 && dz32 > -(1 << 23) && dz32 < (1 << 23)) {   // uniform; full-rate products
                q.x += __mul24(J[0], dz32);
                q.y += __mul24(J[1], dz32);
                q.z += __mul24(J[2], dz32);
                q.w += __mul24(J[3], dz32);
            } else {
                q.x = (int32_t)((uint32_t)q.x + (uint32_t)J[0] * (uint32_t)dz32);
                q.y = (int32_t)((uint32_t)q.y + (uint32_t)J[1] * (uint32_t)dz32);
                q.z = (int32_t)((uint32_t)q.z + (uint32_t)J[2] * (uint32_t)dz32);
                q.w = (int32_t)((uint32_t)q.w + (uint32_t)J[3] * (uint32_t)dz32);
            }
            *(int4 *)&c1[j0] = q;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                c1[j0 + u] = (C)((uint64_t)c1[j0 + u] + (uint64_t)(int64_t)J[u] * (uint64_t)dz);
        }
    }
}

// A heat-bath draw by enumeration, by the whole team: value j of the range belongs to thread j / c,
// c = ceil(W / nthr) <= 4.  inv = -1 / (2 a2) (a2 > 0).  Two barriers (four where single precision cannot
// decide); every thread returns the drawn value.
// Weights are relative to the smallest dE, that of vm: an end of the range, or (a2 > 0) one of the two
// integers around the vertex -a1 / (2 a2), whose computed value errs by less than would move it past an
// integer that is not the minimum itself; dE(v) - dE(vm) = (v - vm) (a1 + a2 (v + vm)), an exact integer.
template <bool kSmall>
__device__ __forceinline__ int64_t team_draw(int64_t a1, int64_t a2, double inv, int64_t lo, int64_t W, double beta, double U,
                                             bool exact53, int lane, int wave, int tid, int nthr, TeamExchange *X, int turn,
                                             ScanCarry &cy) {
    constexpr int kMost = 4;
    const int64_t hi = lo + W - 1;
    auto rise = [&](int64_t v, int64_t from) -> int64_t {
        if (kSmall) {
            const int32_t dv = (int32_t)v - (int32_t)from, sv = (int32_t)v + (int32_t)from;
            return ((int64_t)(int32_t)a1 + (int64_t)(int32_t)a2 * (int64_t)sv) * (int64_t)dv;
        }
        return (v - from) * (a1 + a2 * (v + from));
    };
    int64_t vm = rise(hi, lo) < 0 ? hi : lo;
    if (a2 > 0) {   // uniform
        const double t = (double)a1 * inv;
        const int64_t f = t < (double)lo ? lo : t > (double)hi ? hi : (int64_t)__builtin_floor(t);
        const int64_t g = f < hi ? f + 1 : hi;
        vm = rise(g, f) < 0 ? g : f;
    }
    const uint32_t W32 = (uint32_t)W;
    const uint32_t c = (W32 + (uint32_t)nthr - 1u) / (uint32_t)nthr;
    const uint32_t j0 = (uint32_t)tid * c;
    const double a1d = (double)a1, a2d = (double)a2, vmd = (double)vm;
    auto above = [&](uint32_t j) -> double {   // value j's energy above the minimum
        const int64_t v = lo + (int64_t)j;
        if (exact53) {   // every product and sum below 2^53
            const double vd = (double)(int32_t)v;
            return (vd - vmd) * fma(a2d, vd + vmd, a1d);
        }
        return (double)rise(v, vm);
    };
    const int nw = nthr / kWave;
    {
        // In single precision first, as draw_single: at most four additions per lane, six in the scan and
        // four in the waves' scan, <t> <= ln 4096 = 8.4, so below 5.5e-6 of the total; the margin is 1.2e-5.
        // Only the wave that holds the threshold decides: cumulative weights never decrease, so where its
        // first and last are clear of the threshold the other waves' are too.
        const float kf = (float)(beta * -1.4426950408889634);
        float f[kMost], sum = 0.0f;
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
            f[i] = 0.0f;
            if ((uint32_t)i < c) {   // uniform
                const uint32_t j = j0 + (uint32_t)i;
                const float e = __builtin_amdgcn_exp2f(kf * (float)above(j < W32 ? j : W32 - 1u));
                f[i] = j < W32 ? e : 0.0f;
                sum += f[i];
            }
        }
        const float incl = wave_scan_f32(sum);
        if (lane == kWave - 1) X->sum[turn][wave] = (double)incl;
        window_barrier();
        const float ws = wave_scan_f32(lane < nw ? (float)X->sum[turn][lane] : 0.0f);
        auto of = [&](float x, int l) { return __uint_as_float(lane_read32(__float_as_uint(x), l)); };
        const float total = of(ws, nw - 1), thr = (float)U * total, tol = 1.2e-5f * total;
        const uint64_t past = __ballot(lane < nw && ws > thr);
        const int holder = past ? __ffsll((unsigned long long)past) - 1 : nw - 1;
        if (wave == holder) {
            const float first = wave > 0 ? of(ws, wave - 1) : 0.0f;
            float run = first + __uint_as_float(dpp32<0x138, 0xf, 0xf>(__float_as_uint(incl), 0));
            int32_t hit = -1;
            bool near = wave > 0 && !(__builtin_fabsf(first - thr) > tol);
#pragma unroll
            for (int i = 0; i < kMost; ++i) {
                run += f[i];
                const bool in = (uint32_t)i < c && j0 + (uint32_t)i < W32;
                near = near || (in && !(__builtin_fabsf(run - thr) > tol));
                hit = hit < 0 && in && run > thr ? (int32_t)(j0 + (uint32_t)i) : hit;
            }
            const uint64_t m = __ballot(hit >= 0);
            const bool sure = m != 0 && __ballot(near) == 0;
            const int32_t j = m ? (int32_t)lane_read32((uint32_t)hit, __ffsll((unsigned long long)m) - 1) : 0;
            if (lane == 0) X->drawn[turn] = sure ? j : -1;
        }
        window_barrier();
        const int32_t j = X->drawn[turn];
        if (j >= 0) return lo + (int64_t)j;   // uniform over the team
    }
    double w[kMost], lane_sum = 0.0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        w[i] = 0.0;
        if ((uint32_t)i < c) {   // uniform
            const uint32_t j = j0 + (uint32_t)i;
            const double e = exp_nonpos(-(beta * above(j < W32 ? j : W32 - 1u)));
            w[i] = j < W32 ? e : 0.0;
            lane_sum += w[i];
        }
    }
    const double incl = wave_scan_rows(lane_sum, cy);
    if (lane == kWave - 1) X->sum[turn][wave] = incl;
    window_barrier();
    // every wave: the running sums of the waves' sums, in lanes 0 .. 15
    const double ws = wave_scan_rows(lane < nw ? X->sum[turn][lane] : 0.0, cy);
    const double thr = U * lane_double(ws, nw - 1);
    const uint64_t past = __ballot(lane < nw && ws > thr);
    const int holder = past ? __ffsll((unsigned long long)past) - 1 : nw - 1;   // the wave that holds the drawn value
    if (wave == holder) {
        const double before = (wave > 0 ? lane_double(ws, wave - 1) : 0.0) + wave_shift_up1_zero(incl, cy);
        double run = 0.0;
        int32_t hit = -1;
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
            run += w[i];
            const bool pass = (uint32_t)i < c && j0 + (uint32_t)i < W32 && before + run > thr;
            hit = hit < 0 && pass ? i : hit;
        }
        const uint64_t m = __ballot(hit >= 0);
        uint32_t j;   // (where rounding leaves no value past the threshold, the wave's last)
        if (m) {
            const int src = __ffsll((unsigned long long)m) - 1;
            j = ((uint32_t)wave * kWave + (uint32_t)src) * c + lane_read32((uint32_t)hit, src);
        } else {
            j = ((uint32_t)wave + 1u) * kWave * c - 1u;
        }
        if (lane == 0) X->drawn[turn] = (int32_t)(j < W32 ? j : W32 - 1u);
    }
    window_barrier();
    return lo + (int64_t)X->drawn[turn];
}

// The sweeps of one replica by its team.  Returns in E the energy changes (the same in every thread).
template <int kRule, typename C, typename ZT>
__device__ __forceinline__ void team_sweeps(const TeamCtx &T, ZT *z, C *c1, TeamExchange *X, int64_t &E) {
    const DevProblem &P = T.P;
    const int32_t n = P.n;
    const int lane = T.tid & (kWave - 1), wave = T.tid / kWave;
    constexpr bool kHeatBath = kRule == SA_HEAT_BATH;
    const bool closed = kHeatBath && T.closed;
    constexpr bool kSmallC = sizeof(C) == 4;   // c1 and the values fit 32 bits
    ScanCarry cy;
    int turn = 0;
    bool hot = true;   // the last block changed at least a quarter of its variables
    auto load = [&](int32_t b) {
        SchedRec m;
        if (b + lane < n) {
            m = T.order[b + lane];
        } else {
            m.k = -1;
            m.lo = 0;
            m.width = 1;
            m.emask = 0;
        }
        return m;
    };
    for (int32_t s = T.s_begin; s < T.s_end; ++s) {
        const double beta = T.beta[s];
        const double r_opt =
            T.otm_r >= 0.0 ? T.otm_r : (T.n_sweeps > 1 ? (double)s / (double)(T.n_sweeps - 1) : 0.0);
        uint64_t H = 0;
        SchedRec nx = load(0);
        for (int32_t b = 0; b < n; b += kWave) {
            const SchedRec sl = nx;
            nx = load(b + kWave);
            const bool valid = sl.k >= 0;
            const int32_t kk = valid ? sl.k : 0;
            const int64_t lo = sl.lo, hi = lo + (int64_t)(uint32_t)sl.width - 1;
            const uint32_t W32 = (uint32_t)sl.width;
            const int64_t zk = (int64_t)z[kk];
            const int64_t a2 = valid ? P.d[kk] : 0;
            const bool linear = a2 == 0;
            const double inv = -0.5 / (double)a2;   // (read where a2 > 0)
            const bool all_linear = __ballot(valid && !linear) == 0;
            uint32_t x0 = (uint32_t)sl.k, x1 = (uint32_t)s, x2 = T.read, x3 = T.instance_id;
            philox4x32_10(x0, x1, x2, x3, T.key0, T.key1);
            const double U = (double)((((uint64_t)x2 << 32) | x3) >> 11) * 0x1p-53;
            const uint64_t live = __ballot(valid);
            auto row_of = [&](int j) -> uint2 {   // this thread's couplings of lane j's variable
                uint2 w = make_uint2(0, 0);
                if (P.jbytes != 1 || 4 * T.tid >= n) return w;
                const int32_t k = (int32_t)lane_read32((uint32_t)sl.k, j);
                const int8_t *r = (const int8_t *)P.jd + (size_t)k * P.row_stride + 4 * T.tid;
                w.x = *(const uint32_t *)r;
                if (4 * (T.tid + T.nthr) < n) w.y = *(const uint32_t *)(r + 4 * T.nthr);
                return w;
            };
            uint64_t todo = live;
            int changes = 0;
            uint2 row = make_uint2(0, 0);   // the couplings loaded ahead, of lane row_for's variable
            int row_for = -1;
            while (todo != 0) {   // uniform over the team
                int64_t a1 = (int64_t)c1[kk];
                int want = 2;
                int64_t v = zk, d = 0;
                auto de = [&](int64_t y) -> int64_t {
                    if (kSmallC) {
                        const int32_t dv = (int32_t)y - (int32_t)zk, sv = (int32_t)y + (int32_t)zk;
                        if (all_linear) return (int64_t)(int32_t)a1 * (int64_t)dv;
                        return ((int64_t)(int32_t)a1 + (int64_t)(int32_t)a2 * (int64_t)sv) * (int64_t)dv;
                    }
                    return (y - zk) * (a1 + a2 * (y + zk));
                };
                auto margin = [&]() -> double {   // as in settled_block
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
                    return (double)m;
                };
                if (!kHeatBath) {
                    if (kRule == SA_OPT_METROPOLIS && (double)x0 * 0x1p-32 < r_opt) {
                        v = linear ? (a1 >= 0 ? lo : hi) : margin() > 0.0 ? zk : lane_argmin_quadratic(a1, a2, lo, hi, zk);
                    } else {
                        v = lo + (int64_t)(((uint64_t)x1 * (uint64_t)(W32 - 1u)) >> 32);
                        if (v >= zk) v += 1;
                    }
                    d = de(v);
                    want = v != zk && metropolis_accept(d, beta, U) ? 1 : 0;
                } else if (!hot) {
                    if (linear) {
                        // (its rare double-precision rest out of line: inlined, it spilled registers of the hot
                        // draws, N = 4096, W = 2001, 20 sweeps x 16 reads 100.4 to 102.1 ms)
                        v = closed ? heat_bath_closed(a1, lo, (int64_t)W32, beta, U, x1)
                                   : linear_draw<true>(a1, lo, W32, beta, U);
                        d = de(v);
                        want = v != zk ? 1 : 0;
                    } else {
                        const double M = margin();
                        if (M > 0.0) {
                            const double ex = exp_nonpos(-(beta * M));
                            const double rho = a2 >= 0 ? 2.0 * geometric_tail(ex) : (double)(W32 - 1u) * ex;
                            want = heat_bath_stays(rho, U) ? 0 : 2;
                        }
                    }
                }
                uint64_t mask = __ballot(valid && want != 0) & todo;
                bool changed = false;
                while (mask != 0 && !changed) {   // uniform
                    const int j = __ffsll((unsigned long long)mask) - 1;
                    mask &= mask - 1;
                    todo = j == kWave - 1 ? 0ull : live & (~0ull << (j + 1));
                    const uint2 row_j = row_for == j ? row : row_of(j);
                    const int32_t kj = (int32_t)lane_read32((uint32_t)sl.k, j);
                    // the next row, under this draw (where this variable changes, another lane may be
                    // served next, and its row is loaded then)
                    const uint64_t after = hot ? todo : mask;
                    if (after != 0) {
                        row_for = __ffsll((unsigned long long)after) - 1;
                        row = row_of(row_for);
                    }
                    const int64_t zj = (int64_t)(int32_t)lane_read32((uint32_t)(int32_t)zk, j);
                    int64_t vj, dj;
                    bool apart = true;   // a barrier lies between the waves' reads of c1 and its update
                    if (lane_read32((uint32_t)want, j) == 1u) {
                        apart = false;
                        vj = (int64_t)(int32_t)lane_read32((uint32_t)(int32_t)v, j);
                        dj = (int64_t)lane_read64((uint64_t)d, j);
                    } else {
                        const int64_t loj = (int32_t)lane_read32((uint32_t)sl.lo, j);
                        const int64_t Wj = (int64_t)lane_read32((uint32_t)sl.width, j);
                        const double Uj = lane_double(U, j);
                        const int64_t a1j = (int64_t)lane_read64((uint64_t)a1, j);
                        const int64_t a2j = (int64_t)lane_read64((uint64_t)a2, j);
                        if (a2j == 0) {
                            vj = closed ? heat_bath_closed(a1j, loj, Wj, beta, Uj, lane_read32(x1, j))
                                        : linear_draw(a1j, loj, (uint32_t)Wj, beta, Uj);
                            apart = false;
                        } else {
                            vj = team_draw<kSmallC>(a1j, a2j, lane_double(inv, j), loj, Wj, beta, Uj, T.exact53, lane, wave, T.tid,
                                           T.nthr, X, turn, cy);
                            turn ^= 1;
                        }
                        if (kSmallC)
                            dj = ((int64_t)(int32_t)a1j + (int64_t)(int32_t)a2j * (int64_t)((int32_t)vj + (int32_t)zj)) *
                                 (int64_t)((int32_t)vj - (int32_t)zj);
                        else
                            dj = (vj - zj) * (a1j + a2j * (vj + zj));
                    }
                    changed = vj != zj;
                    if (changed) {
                        changes += 1;
                        E += dj;
                        if (T.trace) H += hash_word(kj, vj) - hash_word(kj, zj);
                        if (!apart) window_barrier();
                        team_update(P, c1, kj, vj - zj, T.tid, T.nthr, row_j);
                        if (T.tid == 0) z[kj] = (ZT)vj;   // (read again a sweep on, after barriers)
                        window_barrier();
                    }
                }
                if (!changed) break;
            }
            hot = changes >= 16;
        }
        if (T.trace && H != 0 && T.tid == 0) atomicAdd((unsigned long long *)&T.trace[s], (unsigned long long)H);
        window_barrier();   // z before the next sweep's reads
    }
}

// c1 of every variable from the state: one row per wave at a time.
template <typename C, typename ZT>
__device__ __forceinline__ void team_init(const DevProblem &P, const ZT *z, C *c1, int tid, int nthr) {
    const int lane = tid & (kWave - 1);
    for (int32_t k = tid / kWave; k < P.n; k += nthr / kWave) {
        using Ring = std::conditional_t<sizeof(C) == 4, uint32_t, uint64_t>;
        const Ring a = wave_sum<Ring>(dense_dot<Ring, ZT>(P, z, k, lane, nullptr)) + (Ring)P.h[k];
        if (lane == 0) c1[k] = (C)a;
    }
    for (int32_t k = P.n + tid; k < P.row_stride; k += nthr) c1[k] = 0;
}

// E(z) = sum_k z_k (h_k + d_k z_k) + 1/2 sum_k z_k (c1_k - h_k) (every pair is in two of the last sum's
// terms, and twice the pairs' energy fits int64), summed over the team; z and c1 complete.
template <typename C, typename ZT>
__device__ __forceinline__ int64_t team_energy(const DevProblem &P, const ZT *z, const C *c1, TeamExchange *X, int tid, int nthr) {
    uint64_t once = 0, twice = 0;
    for (int32_t k = tid; k < P.n; k += nthr) {
        const int64_t v = z[k];
        once += (uint64_t)(v * (P.h[k] + P.d[k] * v));
        twice += (uint64_t)(v * ((int64_t)c1[k] - P.h[k]));
    }
    once = wave_sum_u64(once);
    twice = wave_sum_u64(twice);
    if ((tid & (kWave - 1)) == 0) {
        X->sum[0][tid / kWave] = __longlong_as_double((long long)once);
        X->sum[1][tid / kWave] = __longlong_as_double((long long)twice);
    }
    window_barrier();
    uint64_t a = 0, b = 0;
    for (int w = 0; w < nthr / kWave; ++w) {
        a += (uint64_t)__double_as_longlong(X->sum[0][w]);
        b += (uint64_t)__double_as_longlong(X->sum[1][w]);
    }
    window_barrier();
    return (int64_t)a + (int64_t)b / 2;
}

// Plain runs: one workgroup per read.
template <int kRule, typename C>
__global__ void __launch_bounds__(1024) dense_team_kernel(AnnealArgs A) {
    extern __shared__ int32_t lds_state[];
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const int read = (int)blockIdx.x;
    if (read >= A.n_reads) return;
    const int32_t n = A.P.n;
    TeamExchange *X = (TeamExchange *)lds_state;
    C *c1 = (C *)((char *)lds_state + A.off_c);
    int32_t *z = (int32_t *)((char *)lds_state + A.off_m);
    init_state(A.P, z, A.z_init ? A.z_init + (size_t)read * n : nullptr, (uint32_t)read, A.instance_id, A.key0, A.key1, tid,
               nthr);
    window_barrier();
    TeamCtx T;
    T.P = A.P;
    T.beta = A.beta;
    T.n_sweeps = A.n_sweeps;
    T.s_begin = A.s_begin;
    T.s_end = A.s_end;
    T.key0 = A.key0;
    T.key1 = A.key1;
    T.instance_id = A.instance_id;
    T.read = (uint32_t)read;
    T.otm_r = A.otm_r;
    T.order = A.order;
    T.closed = A.closed != 0;
    T.exact53 = A.exact53 != 0;
    T.tid = tid;
    T.nthr = nthr;
    uint64_t *trace = A.trace ? A.trace + (size_t)read * (size_t)(A.s_end - A.s_begin) : nullptr;
    T.trace = trace ? trace - A.s_begin : nullptr;
    if (trace && A.s_end > A.s_begin) {
        uint64_t h0 = 0;
        for (int32_t k = tid; k < n; k += nthr) h0 += hash_word(k, z[k]);
        h0 = wave_sum_u64(h0);
        if ((tid & (kWave - 1)) == 0) atomicAdd((unsigned long long *)&trace[0], (unsigned long long)h0);
    }
    team_init(A.P, z, c1, tid, nthr);
    window_barrier();
    int64_t E = team_energy(A.P, z, c1, X, tid, nthr);
    team_sweeps<kRule, C, int32_t>(T, z, c1, X, E);
    int32_t *zo = A.z_out + (size_t)read * n;
    for (int32_t k = tid; k < n; k += nthr) zo[k] = z[k];
    if (tid == 0) A.e_out[read] = E;
}

// Batches and server chunks: task blockIdx.x, sweeps s_begin .. s_end of one read.
template <int kRule, typename C>
__global__ void __launch_bounds__(1024) dense_team_batch_kernel(const BatchInst *insts, const BatchTask *tasks) {
    extern __shared__ int32_t lds_state[];
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const BatchTask task = tasks[blockIdx.x];
    const BatchInst &D = insts[task.inst];
    const int32_t read = task.read;
    TeamExchange *X = (TeamExchange *)lds_state;
    C *c1 = (C *)((char *)lds_state + D.off_c);
    int32_t *z = (int32_t *)((char *)lds_state + D.off_m);
    TeamCtx T;
    T.P = D.P;
    const int32_t n = T.P.n;
    int32_t *zo = D.z_out + (size_t)read * n;
    init_state(T.P, z, D.resume ? zo : nullptr, (uint32_t)read, D.instance_id, D.key0, D.key1, tid, nthr);
    window_barrier();
    T.beta = D.beta;
    T.n_sweeps = D.n_sweeps;
    T.s_begin = D.s_begin;
    T.s_end = D.s_end;
    T.key0 = D.key0;
    T.key1 = D.key1;
    T.instance_id = D.instance_id;
    T.read = (uint32_t)read;
    T.otm_r = -1.0;
    T.order = D.order;
    T.closed = D.rule == SA_HEAT_BATH_CLOSED;
    T.exact53 = D.exact53 != 0;
    T.tid = tid;
    T.nthr = nthr;
    T.trace = nullptr;
    team_init(T.P, z, c1, tid, nthr);
    window_barrier();
    int64_t E = D.resume ? D.e_out[read] : team_energy(T.P, z, c1, X, tid, nthr);
    team_sweeps<kRule, C, int32_t>(T, z, c1, X, E);
    for (int32_t k = tid; k < n; k += nthr) zo[k] = z[k];
    if (tid == 0) D.e_out[read] = E;
}

}  // namespace
}  // namespace sa
