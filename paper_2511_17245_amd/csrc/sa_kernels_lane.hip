// sa_kernels_lane.hip -- launch of the lane kernel (sa_lane.h).
#include <algorithm>
#include <type_traits>

#include "sa_lane.h"

namespace sa {

bool lane_eligible(int rule, const Packed &p, bool coef32, int device, bool &compact) {
    compact = false;
    if ((rule != SA_HEAT_BATH && rule != SA_HEAT_BATH_CLOSED) || p.dense || p.pair_row.empty()) return false;
    int max_lds = 65536;
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
    if (shared_state_bytes(p.n, kLaneMaxWaves) > max_lds) return false;
    compact = coef32 && p.z23 && p.n <= 65536;
    for (size_t i = 0; compact && i < p.pair.size(); ++i) compact = p.pair[i].J >= INT16_MIN && p.pair[i].J <= INT16_MAX;
    return true;
}

int32_t lane_off_places(int32_t n, int waves) { return (int32_t)((shared_state_bytes(n, waves) + 15) & ~(int64_t)15); }

int64_t lane_lds_bytes(int32_t n, int waves, int32_t n_rounds) {
    return lane_off_places(n, waves) + 16 * (int64_t)n_rounds * waves;
}

int lane_waves(const LaneImage &im, int32_t n, int32_t n_reads, int device) {
    // a level of fewer than eight variables leaves a wave's lanes idle that the windows would use
    if (im.n_levels <= 0 || (int64_t)im.n_slots < 8 * (int64_t)im.n_levels) return 0;
    int cus = 256, max_lds = 65536;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
    // a wave for every chunk of an average level, as far as all replicas' waves are resident (two per SIMD)
    // and the places fit
    const int32_t chunks = im.level_chunk.back();
    const int32_t mean = (chunks + im.n_levels - 1) / im.n_levels;
    auto fits = [&](int w) { return lane_lds_bytes(n, w, im.n_levels + chunks / w) <= max_lds; };
    if (!fits(1)) return 0;
    int waves = 1;
    while (waves < kLaneMaxWaves && waves < mean && fits(2 * waves) && (int64_t)n_reads * waves * 2 <= (int64_t)cus * 8)
        waves *= 2;
    return waves;
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
