// sa_kernels_lane.hip -- launch of the lane kernel (sa_lane.h).
#include <algorithm>
#include <type_traits>

#include "sa_lane.h"

namespace sa {

bool lane_eligible(int rule, const Packed &p, bool coef32, int max_lds, bool &compact) {
    compact = false;
    if ((rule != SA_HEAT_BATH && rule != SA_HEAT_BATH_CLOSED) || p.dense || p.pair_row.empty()) return false;
    if (lane_off_places(p.n, kLaneMaxWaves) > max_lds) return false;
    compact = coef32 && p.z23 && p.pair16;
    return true;
}

int launch_lane(LaneArgs a, bool compact, int waves, void *stream, std::string &err) {
    using Fn = void (*)(LaneArgs);
    a.off_places = lane_off_places(a.P.n, waves);
    Fn fn = compact ? (Fn)lane_kernel<true> : (Fn)lane_kernel<false>;
    const int lds = (int)lane_lds_bytes(a.P.n, waves, a.n_rounds);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)a.n_reads), dim3((unsigned)(waves * kWave)), (size_t)lds, (hipStream_t)stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

void group_lanes(const std::vector<LaneChoice> &choices, const std::vector<int32_t> &n_reads, std::vector<BatchTask> &tasks,
                 std::vector<LaneGroup> &groups) {
    groups.clear();
    for (int waves = kLaneMaxWaves; waves >= 1; waves /= 2) {
        for (int compact = 1; compact >= 0; --compact) {
            LaneGroup g;
            g.first = (int32_t)tasks.size();
            g.waves = waves;
            g.compact = compact != 0;
            for (size_t i = 0; i < choices.size(); ++i) {
                if (choices[i].waves != waves || choices[i].compact != g.compact) continue;
                g.lds_bytes = std::max(g.lds_bytes, choices[i].lds_bytes);
                for (int32_t r = 0; r < n_reads[i]; ++r) tasks.push_back(BatchTask{(int32_t)i, r});
            }
            g.n = (int32_t)tasks.size() - g.first;
            if (g.n > 0) groups.push_back(g);
        }
    }
}

int launch_lane_group(const LaneArgs *list, const BatchTask *tasks, const LaneGroup &g, void *stream, std::string &err) {
    using Fn = void (*)(const LaneArgs *, const BatchTask *);
    Fn fn = g.compact ? (Fn)lane_batch_kernel<true> : (Fn)lane_batch_kernel<false>;
    if (g.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, g.lds_bytes);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)g.n), dim3((unsigned)(g.waves * kWave)), (size_t)g.lds_bytes, (hipStream_t)stream,
                       list, tasks + g.first);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("kernel launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return SA_OK;
}

}  // namespace sa
