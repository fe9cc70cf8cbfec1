// sa_kernels_settled.hip -- variants and launch of the settled kernel (sa_settled.h).
#include <algorithm>

#include "sa_settled.h"

namespace sa {
namespace {

using SettledFn = void (*)(AnnealArgs);

// Heat-bath visits: weights per lane in registers up to 8 (kRegChunk), recomputed above.
template <bool kDense, int kRule, int kMaxE, typename Acc>
SettledFn pick_chunk(int32_t max_width) {
    if (max_width <= kWave) return settled_kernel<kDense, kRule, 1, kMaxE, Acc>;
    if (max_width <= 8 * kWave) return settled_kernel<kDense, kRule, 8, kMaxE, Acc>;
    return settled_kernel<kDense, kRule, 0, kMaxE, Acc>;
}

template <bool kDense, int kMaxE, typename Acc>
SettledFn pick_rule(int rule, int32_t max_width, int32_t otm_enum_max) {
    switch (rule) {
        case SA_METROPOLIS: return settled_kernel<kDense, SA_METROPOLIS, 0, 1, Acc>;
        case SA_HEAT_BATH: return pick_chunk<kDense, SA_HEAT_BATH, kMaxE, Acc>(max_width);
        case SA_HEAT_BATH_CLOSED: return pick_chunk<kDense, SA_HEAT_BATH_CLOSED, kMaxE, Acc>(max_width);
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
    int cus = 256, max_lds = 65536;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
    const int64_t n = p.n, state = (4 * n + 7) & ~(int64_t)7;
    // the dense form changes every cached sum with each move: no gain beyond the sizes that keep the
    // cache in the ordinary kernel too
    if (p.dense && n > 1024) return sc;
    const bool sparse_cache = !p.dense && coef32 && p.any_cached;
    const int64_t c = p.dense ? 8 * n : sparse_cache ? state : 0, c2 = sparse_cache && p.any_square ? state : 0;
    const int64_t bytes = state + c + c2 + 2 * ((n + 3) & ~(int64_t)3);
    // every replica at once, or in two goes
    if (bytes > max_lds || (max_lds / bytes) * cus * 2 < n_reads) return sc;
    sc.lds_bytes = (int)bytes;
    sc.off_c = c ? (int)state : -1;
    sc.off_c2 = c2 ? (int)(state + c) : -1;
    sc.off_m = (int)(state + c + c2);
    return sc;
}

int launch_settled(int rule, AnnealArgs a, const SettledChoice &sc, int32_t max_width, int32_t max_exp, bool narrow,
                   void *stream, std::string &err) {
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

int launch_windows(int rule, AnnealArgs a, const LaunchChoice &lc, const SettledChoice &sc, int32_t max_width,
                   int32_t max_exp, bool narrow, void *stream, std::string &err) {
    a.phase = kPhaseWhole;
    if (sc.lds_bytes == 0) return launch_anneal(rule, a, lc, stream, err);
    a.phase = kPhaseFirst;
    a.leave = std::max<int32_t>(1, (int32_t)(3 * (int64_t)a.n_order / settled_share(lc.win_waves)));
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
    q.n_order = a.n_order;
    a.leave = std::max<int32_t>(1, (int32_t)(3 * (int64_t)a.n_order / kSettledShareQuad));
    int rc = launch_quad_mo(rule, q, max_width, max_exp, narrow, stream, err);
    if (rc == SA_OK) rc = launch_settled(rule, a, sc, max_width, max_exp, narrow, stream, err);
    if (rc != SA_OK) return rc;
    q.phase = kPhaseLast;
    q.z_init = q.z_out;
    return launch_quad_mo(rule, q, max_width, max_exp, narrow, stream, err);
}

}  // namespace sa
