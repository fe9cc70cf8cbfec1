// sa_kernels_settled.hip -- variants and launch of the settled kernel (sa_settled.h).
#include <algorithm>

#include "sa_settled.h"

namespace sa {
namespace {

using SettledFn = void (*)(AnnealArgs);

template <bool kDense, int kMaxE, typename Acc>
SettledFn pick_rule(int rule, int32_t max_width, int32_t otm_enum_max) {
    switch (rule) {
        case SA_METROPOLIS: return settled_kernel<kDense, SA_METROPOLIS, 0, 1, Acc>;
        case SA_HEAT_BATH:
        case SA_HEAT_BATH_CLOSED: return settled_kernel<kDense, SA_HEAT_BATH, 0, kMaxE, Acc>;
        default:
            return max_width > otm_enum_max ? settled_kernel<kDense, SA_OPT_METROPOLIS, 1, kMaxE < 4 ? kMaxE : 4, Acc>
                                            : settled_kernel<kDense, SA_OPT_METROPOLIS, 0, kMaxE < 4 ? kMaxE : 4, Acc>;
    }
}

}  // namespace

SettledChoice choose_settled(const Packed &p, bool coef32, int32_t n_reads, int32_t n_order, int32_t n_sweeps, int device) {
    SettledChoice sc;
    // a run too short to gain what two more launches cost (about 10 us; a sweep that changes nothing
    // costs about 0.5 us per variable in the ordinary kernels)
    if (n_sweeps < 16 || (int64_t)n_sweeps * n_order < 2000) return sc;
    // nor one of very few variables.  (The line was drawn when each replica left by itself and N = 21 binary
    // variables that keep changing lost, 4.3 to 5.5 ms.  They leave together now, and from 8 variables on no run
    // of any rule was slower than 0.98 times with the line at 1: 360 runs of 8 to 23 variables of 2 to 101
    // values, 300 to 3000 sweeps, the best seven times as fast.)
    if (n_order < 24) return sc;
    int cus = 256, max_lds = 65536;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
    const int64_t n = p.n, state = (4 * n + 7) & ~(int64_t)7;
    // the dense form changes every cached sum with each move: no gain beyond the sizes that keep the
    // cache in the ordinary kernel too
    if (p.dense && n > 1024) return sc;
    const bool sparse_cache = !p.dense && p.any_cached;
    const int64_t words = coef32 ? state : 8 * n;
    const int64_t c = p.dense ? 8 * n : sparse_cache ? words : 0, c2 = sparse_cache && p.any_square ? words : 0;
    const int64_t bytes = state + c + c2 + 2 * ((n + 3) & ~(int64_t)3);
    // Every replica at once, or in two goes, for pair problems in 1.8, as the quad kernel's sweep of them is no
    // dearer than two settled ones: with against without, 200 sweeps, HUIO N = 4000 at 1.9 goes 48.7 and 53.4 ms
    // (Metropolis), 51.6 and 57.0 (optimal transition), at 2.2 71.1 and 65.7, 95.7 and 109.1; pairs, 500 sweeps, W = 17,
    // N = 6000 at 1.76 goes 163.8 and 169.9, 159.6 and 165.9, N = 10000 at 2 196.7 and 188.7, 211.6 and 196.2.
    // (The windows gain at up to 4.5 goes: dense N = 1000, Metropolis 1222 and 1426, N = 200 401 and 412.)
    const int64_t tenths = p.pair_row.empty() ? 20 : 18;
    if (bytes > max_lds || (max_lds / bytes) * cus * tenths / 10 < n_reads) return sc;
    sc.lds_bytes = (int)bytes;
    sc.off_c = c ? (int)state : -1;
    sc.off_c2 = c2 ? (int)(state + c) : -1;
    sc.off_m = (int)(state + c + c2);
    return sc;
}

int launch_settled(int rule, AnnealArgs a, const SettledChoice &sc, int32_t max_width, int32_t max_exp, bool narrow,
                   void *stream, std::string &err) {
    a.closed = rule == SA_HEAT_BATH_CLOSED ? 1 : 0;
    a.off_c = sc.off_c;
    a.off_c2 = sc.off_c2;
    a.off_m = sc.off_m;
    const int cls = maxe_class_of(max_exp);
    if (rule == SA_OPT_METROPOLIS && max_width > a.otm_enum_max) narrow = false;   // as launch_anneal
    SettledFn fn;
    if (a.P.dense) {
        if (cls == 1)
            fn = narrow ? pick_rule<true, 1, uint32_t>(rule, max_width, a.otm_enum_max)
                        : pick_rule<true, 1, uint64_t>(rule, max_width, a.otm_enum_max);
        else
            fn = narrow ? pick_rule<true, 2, uint32_t>(rule, max_width, a.otm_enum_max)
                        : pick_rule<true, 2, uint64_t>(rule, max_width, a.otm_enum_max);
    } else if (cls == 1) {
        fn = narrow ? pick_rule<false, 1, uint32_t>(rule, max_width, a.otm_enum_max)
                    : pick_rule<false, 1, uint64_t>(rule, max_width, a.otm_enum_max);
    } else if (cls == 2) {
        fn = narrow ? pick_rule<false, 2, uint32_t>(rule, max_width, a.otm_enum_max)
                    : pick_rule<false, 2, uint64_t>(rule, max_width, a.otm_enum_max);
    } else if (cls == 4) {
        fn = pick_rule<false, 4, uint64_t>(rule, max_width, a.otm_enum_max);
    } else {
        fn = pick_rule<false, kMaxExpPoly, uint64_t>(rule, max_width, a.otm_enum_max);
    }
    if (sc.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, sc.lds_bytes);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)a.n_reads), dim3(kWave), (size_t)sc.lds_bytes, (hipStream_t)stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

int launch_windows(int rule, AnnealArgs a, const LaunchChoice &lc, const SettledChoice &sc, int32_t share, int32_t max_width,
                   int32_t max_exp, bool narrow, void *stream, std::string &err) {
    a.phase = kPhaseWhole;
    if (sc.lds_bytes == 0) return launch_anneal(rule, a, lc, stream, err);
    a.phase = kPhaseFirst;
    a.every = settled_every(a.n_order, lc.win_waves);
    a.limit = settled_limit(a.n_order, a.every, share);
    int rc = launch_anneal(rule, a, lc, stream, err);
    if (rc == SA_OK) rc = launch_settled(rule, a, sc, max_width, max_exp, narrow, stream, err);
    if (rc != SA_OK) return rc;
    a.phase = kPhaseLast;
    a.z_init = a.z_out;
    return launch_anneal(rule, a, lc, stream, err);
}

int launch_rounds(int rule, QuadArgs q, AnnealArgs a, const SettledChoice &sc, int32_t max_width, int32_t max_exp,
                  bool narrow, void *stream, std::string &err) {
    q.phase = kPhaseWhole;
    if (sc.lds_bytes == 0) return launch_quad_mo(rule, q, max_width, max_exp, narrow, stream, err);
    q.phase = kPhaseFirst;
    a.every = kSettledEveryQuad;
    q.limit = a.limit = settled_limit(a.n_order, a.every, settled_share_quad(q.P.pair != nullptr));
    q.all = a.all;
    int rc = launch_quad_mo(rule, q, max_width, max_exp, narrow, stream, err);
    if (rc == SA_OK) rc = launch_settled(rule, a, sc, max_width, max_exp, narrow, stream, err);
    if (rc != SA_OK) return rc;
    q.phase = kPhaseLast;
    q.z_init = q.z_out;
    return launch_quad_mo(rule, q, max_width, max_exp, narrow, stream, err);
}

int launch_settled_batch(const BatchInst *insts, const BatchTask *tasks, int32_t n_tasks, int lds_bytes, int maxe_class,
                         void *stream, std::string &err) {
    using Fn = void (*)(const BatchInst *, const BatchTask *);
    Fn fn = maxe_class <= 2 ? (Fn)settled_batch_kernel<2>
            : maxe_class <= 4 ? (Fn)settled_batch_kernel<4> : (Fn)settled_batch_kernel<kMaxExpPoly>;
    if (lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)n_tasks), dim3(kWave), (size_t)lds_bytes, (hipStream_t)stream, insts, tasks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

void settle_batch(const std::vector<BatchInst> &insts, const std::vector<int> &lds, const std::vector<double> &cost,
                  std::vector<BatchTask> &tasks, SettledGroup (&groups)[kSettledGroups]) {
    const int limit[kSettledGroups] = {160 * 1024, 40 * 1024, 10 * 1024};
    std::vector<int32_t> order;
    for (size_t i = 0; i < insts.size(); ++i)
        if (lds[i] > 0) order.push_back((int32_t)i);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return cost[(size_t)x] > cost[(size_t)y]; });
    tasks.clear();
    for (int g = 0; g < kSettledGroups; ++g) {
        groups[g] = SettledGroup();
        groups[g].first = (int32_t)tasks.size();
        for (int32_t i : order) {
            const int b = lds[(size_t)i];
            if (b > limit[g] || (g + 1 < kSettledGroups && b <= limit[g + 1])) continue;
            groups[g].lds_bytes = std::max(groups[g].lds_bytes, b);
            for (int32_t r = 0; r < insts[(size_t)i].n_reads; ++r) tasks.push_back(BatchTask{i, r});
        }
        groups[g].n = (int32_t)tasks.size() - groups[g].first;
    }
}

int settle_inst(const Packed &p, bool coef32, const SchedRec *order, int32_t n_order, int32_t n_sweeps, int device,
                BatchInst &d) {
    d.next = nullptr;
    const SettledChoice sc = choose_settled(p, coef32, 1, n_order, n_sweeps, device);
    if (sc.lds_bytes == 0) return 0;
    d.order = order;
    d.n_order = n_order;
    d.off_c = sc.off_c;
    d.off_c2 = sc.off_c2;
    d.off_m = sc.off_m;
    d.z30 = p.z30 ? 1 : 0;
    d.every = d.limit = 0;   // set with the team size
    return sc.lds_bytes;
}

}  // namespace sa
