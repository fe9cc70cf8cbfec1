// sa_lane.h -- the heat-bath sweep of multilinear pair problems (compact pair records) with one update
// per lane, over the dependency levels of the sweep.
//
// A variable of such a problem has dE(v) = a (v - z_k), and the heat bath's distribution over its range is
// geometric: the draw by enumeration, the first value whose cumulative weight exceeds U times the
// total, is the inverse of the cumulative distribution in closed form (Sec. 3.3.2, multilinear case)
// wherever rounding does not decide.  linear_draw computes that inverse, first in single precision with
// a bound on its error, which decides all but about a part in 10^5 W of the draws; where a step of the
// distribution lies within the bound, in double precision; and where it lies so near that double rounding
// could decide (a part in 10^10), it adds the weights one by one in value order, as the oracle does.  So a
// draw takes one lane some forty instructions whatever the width, where a quad's four lanes evaluated
// W weights, and a wave holds 64 updates instead of 16.
//
// A workgroup anneals one replica, its state in LDS.  The levels (build_levels) follow one another with a
// barrier between; a level's variables are cut into chunks of 64, by falling degree, one chunk per wave
// and round.  A chunk's slots and records are stored lane by lane (record r of lane l at r 64 + l of the
// chunk's rows), so their loads are coalesced; they hold no state, so a wave loads a chunk's slots two
// rounds ahead and its first kLaneAhead records one round ahead, and forms its random words while the
// current chunk's LDS reads are on their way.
//
// What bounds it: the chain of one level (LDS gathers, draw, barrier), about 25 levels per sweep.
// Measured, against the quad kernel: N = 10^4, W = 101, 2000 sweeps x 256 reads 205 to 81 ms; N = 3001 with
// ranges of 2 to 120 values, 400 sweeps x 96 reads 50 to 12 ms.
#pragma once

#include <type_traits>

#include "sa_device.h"

namespace sa {
namespace {

constexpr int kLaneAhead = kLaneReach;   // records of the next chunk loaded one round ahead

// A wave's chunk in one round: the chunk (-1: none; the wave's lanes idle), its first row of records and its
// rows, and whether the round is its level's last.
struct LanePlace {
    int32_t chunk, first, rows, last;
};

// kCompact: records of 16-bit index and coupling, every value below 2^23 and every coefficient below 2^31 in
// magnitude (24-bit products, 32-bit sums); else 32-bit index and coupling and 64-bit sums.
template <bool kCompact>
__device__ __forceinline__ void lane_run(const LaneArgs &A, int read, int32_t *lds_state) {
    using Rec = std::conditional_t<kCompact, uint32_t, uint2>;
    using Sum = std::conditional_t<kCompact, int32_t, int64_t>;
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave, nw = nthr / kWave;
    const int32_t n = A.P.n;
    int32_t *z = lds_state;
    init_state(A.P, z, A.z_init ? A.z_init + (size_t)read * n : nullptr, (uint32_t)read, A.instance_id, A.key0, A.key1, tid,
               nthr);
    window_barrier();
    int64_t E = energy_part(A.P, z, tid, nthr);
    uint64_t *trace = A.trace ? A.trace + (size_t)read * (size_t)(A.s_end - A.s_begin) : nullptr;
    if (trace && A.s_end > A.s_begin) {
        uint64_t h0 = 0;
        for (int32_t k = tid; k < n; k += nthr) h0 += hash_word(k, z[k]);
        h0 = wave_sum_u64(h0);
        if (lane == 0) atomicAdd((unsigned long long *)&trace[0], (unsigned long long)h0);
    }
    // the places of every round and wave, in LDS after the energy parts: read one round before the loads
    // whose addresses they hold
    LanePlace *place = (LanePlace *)((char *)lds_state + A.off_places);
    const int32_t R = A.n_rounds;
    for (int32_t i = tid; i < R * nw; i += nthr) {
        const LaneRows rd = A.rounds[i / nw];   // first chunk, and end (negative: ~end of a level's last round)
        const int32_t end = rd.rows < 0 ? ~rd.rows : rd.rows, c = rd.first + i % nw;
        LanePlace p;
        p.chunk = c < end ? c : -1;
        const LaneRows info = A.chunks[c < end ? c : rd.first];   // (an idle wave loads the round's first chunk)
        p.first = info.first;
        p.rows = c < end ? info.rows : 0;
        p.last = rd.rows < 0 ? 1 : 0;
        place[i] = p;
    }
    window_barrier();
    int64_t dE = 0;
    uint64_t H = 0;
    const bool closed = A.closed != 0;
    if (R > 0 && A.s_end > A.s_begin) {
        auto uniform = [](const LanePlace &q) {
            LanePlace p;
            p.chunk = (int32_t)uni32((uint32_t)q.chunk);
            p.first = (int32_t)uni32((uint32_t)q.first);
            p.rows = (int32_t)uni32((uint32_t)q.rows);
            p.last = (int32_t)uni32((uint32_t)q.last);
            return p;
        };
        auto slot_of = [&](const LanePlace &p) {
            LaneSlot sl = A.slots[(size_t)(p.chunk < 0 ? 0 : p.chunk) * kWave + lane];
            if (p.chunk < 0) sl.k = -1;
            return sl;
        };
        auto load_records = [&](const LanePlace &p, Rec(&r)[kLaneAhead]) {
            const Rec *at = (const Rec *)A.recs + (size_t)(uint32_t)p.first * kWave + lane;
#pragma unroll
            for (int u = 0; u < kLaneAhead; ++u) r[u] = at[(size_t)u * kWave];
        };
        uint32_t x1 = 0, x1n = 0;
        double U = 0.0, Un = 0.0;
        auto words = [&](int32_t k, int32_t s, uint32_t &w1, double &w) {
            uint32_t y0 = (uint32_t)k, y1 = (uint32_t)s, y2 = (uint32_t)read, y3 = A.instance_id;
            uint32_t k0 = A.key0, k1 = A.key1;
            asm volatile("" : "+s"(k0), "+s"(k1));   // (round keys formed again rather than held)
            philox4x32_10(y0, y1, y2, y3, k0, k1);
            w1 = y1;
            w = (double)((((uint64_t)y2 << 32) | y3) >> 11) * 0x1p-53;
        };
        auto after = [&](int32_t r) { return r + 1 < R ? r + 1 : 0; };
        // round r is the current one, rn and rm the next two: pC .. pM their places, slC .. slM their slots
        auto place_at = [&](int32_t r) { return place[r * nw + wave]; };
        LanePlace pC = uniform(place_at(0)), pN = uniform(place_at(after(0))), pM = uniform(place_at(after(after(0))));
        LaneSlot slC = slot_of(pC), slN = slot_of(pN);
        Rec recs[kLaneAhead];
        load_records(pC, recs);
        words(slC.k, A.s_begin, x1, U);
        int32_t rm = after(after(0));
        for (int32_t s = A.s_begin; s < A.s_end; ++s) {
            const double beta = A.beta[s];
            for (int32_t r = 0; r < R; ++r) {   // uniform over the workgroup
                Rec next[kLaneAhead];
                load_records(pN, next);
                const LaneSlot slM = slot_of(pM);
                rm = after(rm);
                const LanePlace pL = place_at(rm);   // (made uniform at the end of the round, when it has arrived)
                const int32_t k = slC.k;
                int32_t zv[kLaneAhead];   // the neighbours' values (an empty record's: variable 0)
                int32_t zk32 = 0;
                if (pC.rows > 0) {
                    zk32 = z[k < 0 ? 0 : k];
#pragma unroll
                    for (int u = 0; u < kLaneAhead; ++u) {
                        if constexpr (kCompact) zv[u] = z[recs[u] & 0xFFFFu];
                        else zv[u] = u < pC.rows ? z[recs[u].x] : 0;
                    }
                }
                words(slN.k, r + 1 < R ? s : s + 1, x1n, Un);   // under those reads
                if (pC.rows > 0) {   // uniform over the wave
                    Sum a = slC.h;
                    auto add = [&](const Rec &q, int32_t v) {
                        if constexpr (kCompact) a += __mul24((int32_t)q >> 16, v);
                        else a += (int64_t)(int32_t)q.y * (int64_t)v;
                    };
#pragma unroll
                    for (int u = 0; u < kLaneAhead; u += 4) {
                        if (u < pC.rows) {   // uniform; rows are whole groups of four
#pragma unroll
                            for (int q = 0; q < 4; ++q) add(recs[u + q], zv[u + q]);
                        }
                    }
                    for (int32_t u = kLaneAhead; u < pC.rows; u += 4) {
                        const Rec *at = (const Rec *)A.recs + (size_t)(uint32_t)(pC.first + u) * kWave + lane;
                        Rec q4[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) q4[q] = at[(size_t)q * kWave];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if constexpr (kCompact) add(q4[q], z[q4[q] & 0xFFFFu]);
                            else add(q4[q], z[q4[q].x]);
                        }
                    }
                    if (k >= 0) {
                        const int64_t zk = zk32, lo = slC.lo;
                        const int64_t v = closed ? heat_bath_closed((int64_t)a, lo, (int64_t)(uint32_t)slC.width, beta, U, x1)
                                                 : linear_draw((int64_t)a, lo, (uint32_t)slC.width, beta, U);
                        if (v != zk) {
                            z[k] = (int32_t)v;
                            dE += (int64_t)a * (v - zk);
                            if (trace) H += hash_word(k, v) - hash_word(k, zk);
                        }
                    }
                }
                if (pC.last) {
                    if (nw > 1) window_barrier();
                    else state_write_fence<true>();
                }
                pC = pN;
                pN = pM;
                pM = uniform(pL);
                slC = slN;
                slN = slM;
                x1 = x1n;
                U = Un;
#pragma unroll
                for (int u = 0; u < kLaneAhead; ++u) recs[u] = next[u];
            }
            if (trace) {
                const uint64_t hw = wave_sum_u64(H);
                if (lane == 0) atomicAdd((unsigned long long *)&trace[s - A.s_begin], (unsigned long long)hw);
                H = 0;
            }
        }
    }
    E += (int64_t)wave_sum_u64((uint64_t)dE);
    int64_t *parts = (int64_t *)(lds_state + (((size_t)n + 1) & ~(size_t)1));
    if (lane == 0) parts[wave] = E;
    window_barrier();
    if (tid == 0) {
        int64_t tot = 0;
        for (int q = 0; q < nw; ++q) tot += parts[q];
        A.e_out[read] = tot;
    }
    int32_t *zo = A.z_out + (size_t)read * n;
    for (int32_t k = tid; k < n; k += nthr) zo[k] = z[k];
}

// Plain runs: one workgroup per read.
template <bool kCompact>
__global__ void __launch_bounds__(512) lane_kernel(LaneArgs A) {
    extern __shared__ int32_t lds_state[];
    if ((int)blockIdx.x >= A.n_reads) return;
    lane_run<kCompact>(A, (int)blockIdx.x, lds_state);
}

// A wave-uniform pointer read from memory, known to point into device memory (a load through a pointer of
// unknown address space counts as an LDS access too, and every wait for LDS would wait for it).
template <typename T>
__device__ __forceinline__ T *in_device_memory(T *p) {
    const uint64_t b = (uint64_t)(uintptr_t)p;
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)(((uint64_t)uni32((uint32_t)(b >> 32)) << 32) |
                                                                  uni32((uint32_t)b));
}

// Batches and server chunks: task blockIdx.x, its problem's arguments in `list`.
template <bool kCompact>
__global__ void __launch_bounds__(512) lane_batch_kernel(const LaneArgs *list, const BatchTask *tasks) {
    extern __shared__ int32_t lds_state[];
    const BatchTask task = tasks[blockIdx.x];
    LaneArgs A = list[task.inst];
    A.P.var = in_device_memory(A.P.var);
    A.P.t_off = in_device_memory(A.P.t_off);
    A.P.t_var = in_device_memory(A.P.t_var);
    A.P.t_coef = in_device_memory(A.P.t_coef);
    A.beta = in_device_memory(A.beta);
    A.rounds = in_device_memory(A.rounds);
    A.chunks = in_device_memory(A.chunks);
    A.slots = in_device_memory(A.slots);
    A.recs = (const void *)in_device_memory((const char *)A.recs);
    if (A.z_init) A.z_init = in_device_memory(A.z_init);
    A.z_out = in_device_memory(A.z_out);
    A.e_out = in_device_memory(A.e_out);
    lane_run<kCompact>(A, task.read, lds_state);
}

}  // namespace
}  // namespace sa
