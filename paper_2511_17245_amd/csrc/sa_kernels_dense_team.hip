// sa_kernels_dense_team.hip -- variants and launch of the dense team kernel (sa_dense_team.h).
#include <algorithm>

#include "sa_dense_team.h"

namespace sa {
namespace {

using TeamFn = void (*)(AnnealArgs);

template <typename C>
TeamFn pick(int rule) {
    switch (rule) {
        case SA_METROPOLIS: return dense_team_kernel<SA_METROPOLIS, C>;
        case SA_OPT_METROPOLIS: return dense_team_kernel<SA_OPT_METROPOLIS, C>;
        default: return dense_team_kernel<SA_HEAT_BATH, C>;
    }
}

}  // namespace

TeamChoice choose_team(int rule, const Packed &p, bool coef32, int32_t n_reads, int device) {
    TeamChoice tc;
    if (!p.dense) return tc;
    int cus = 256, max_lds = 65536;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
    const bool heat_bath = rule == SA_HEAT_BATH || rule == SA_HEAT_BATH_CLOSED;
    // work for the threads: at least two columns of the row (and so many cached sums) or two weights each
    const int64_t work = heat_bath && p.max_exp > 1 ? std::max<int64_t>(p.n, p.max_width) : p.n;
    int waves = 4;
    while (waves < 16 && ((heat_bath && p.max_width > 256 * waves) || p.n > 512 * waves)) waves *= 2;
    if (heat_bath && p.max_width > 256 * waves) return tc;   // (team_draw: at most four values per thread)
    if (128 * (int64_t)waves > work || (int64_t)n_reads * waves > (int64_t)cus * 16) return tc;
    tc.small = coef32 && p.z30;
    tc.exact53 = p.z30 && p.energy_bound < 0x1p50;
    const int64_t c1 = (int64_t)p.row_stride * (tc.small ? 4 : 8);
    const int64_t bytes = kTeamExchangeBytes + c1 + 4 * (int64_t)p.n;
    if (bytes > max_lds) return tc;
    tc.waves = waves;
    tc.off_c = kTeamExchangeBytes;
    tc.off_z = (int)(kTeamExchangeBytes + c1);
    tc.lds_bytes = (int)bytes;
    return tc;
}

int launch_dense_team(int rule, AnnealArgs a, const TeamChoice &tc, void *stream, std::string &err) {
    TeamFn fn = tc.small ? pick<int32_t>(rule) : pick<int64_t>(rule);
    a.closed = rule == SA_HEAT_BATH_CLOSED ? 1 : 0;
    a.exact53 = tc.exact53 ? 1 : 0;
    a.off_c = tc.off_c;
    a.off_m = tc.off_z;
    if (tc.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, tc.lds_bytes);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)a.n_reads), dim3((unsigned)(tc.waves * kWave)), (size_t)tc.lds_bytes,
                       (hipStream_t)stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

TeamChoice team_inst(int rule, const Packed &p, bool coef32, const SchedRec *order, int32_t n_reads, int device, BatchInst &d) {
    const TeamChoice tc = choose_team(rule, p, coef32, n_reads, device);
    d.team_waves = tc.waves;
    if (tc.waves > 0) {
        d.next = nullptr;
        d.order = order;
        d.off_c = tc.off_c;
        d.off_m = tc.off_z;
        d.exact53 = tc.exact53 ? 1 : 0;
    }
    return tc;
}

void group_teams(const std::vector<BatchInst> &insts, const std::vector<TeamChoice> &choices, std::vector<BatchTask> &tasks,
                 std::vector<TeamGroup> &groups) {
    groups.clear();
    std::vector<char> done(insts.size(), 0);
    for (size_t i = 0; i < insts.size(); ++i) {
        if (choices[i].waves == 0 || done[i]) continue;
        TeamGroup g;
        g.first = (int32_t)tasks.size();
        g.rule = insts[i].rule;
        g.waves = choices[i].waves;
        g.small = choices[i].small;
        for (size_t q = i; q < insts.size(); ++q) {
            if (choices[q].waves != g.waves || choices[q].small != g.small || insts[q].rule != g.rule) continue;
            done[q] = 1;
            g.lds_bytes = std::max(g.lds_bytes, choices[q].lds_bytes);
            for (int32_t r = 0; r < insts[q].n_reads; ++r) tasks.push_back(BatchTask{(int32_t)q, r});
        }
        g.n = (int32_t)tasks.size() - g.first;
        groups.push_back(g);
    }
}

int launch_team_group(const BatchInst *insts, const BatchTask *tasks, const TeamGroup &g, void *stream, std::string &err) {
    using Fn = void (*)(const BatchInst *, const BatchTask *);
    Fn fn;
    if (g.small)
        fn = g.rule == SA_METROPOLIS       ? (Fn)dense_team_batch_kernel<SA_METROPOLIS, int32_t>
             : g.rule == SA_OPT_METROPOLIS ? (Fn)dense_team_batch_kernel<SA_OPT_METROPOLIS, int32_t>
                                           : (Fn)dense_team_batch_kernel<SA_HEAT_BATH, int32_t>;
    else
        fn = g.rule == SA_METROPOLIS       ? (Fn)dense_team_batch_kernel<SA_METROPOLIS, int64_t>
             : g.rule == SA_OPT_METROPOLIS ? (Fn)dense_team_batch_kernel<SA_OPT_METROPOLIS, int64_t>
                                           : (Fn)dense_team_batch_kernel<SA_HEAT_BATH, int64_t>;
    if (g.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, g.lds_bytes);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)g.n), dim3((unsigned)(g.waves * kWave)), (size_t)g.lds_bytes, (hipStream_t)stream,
                       insts, tasks + g.first);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

}  // namespace sa
