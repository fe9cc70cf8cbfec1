// sa_kernels_batch.hip -- the persistent batched kernel (many problems in one launch) with 32-bit
// states, and the batched launch.
#include "sa_device.h"
#include "sa_kernel_table.h"

namespace sa {
namespace {

// Sets the batch's task counter to zero (a kernel, so that graph replays stay plain kernel nodes).
__global__ void reset_counter_kernel(uint32_t *counter) {
    if (threadIdx.x == 0) *counter = 0u;
}

}  // namespace

// 32-bit states; 16-bit states are built in sa_kernels_batch16.hip.
BatchKernelFn batch_kernel_z32(int maxe_class, bool narrow) {
    switch (maxe_class) {
        case 1: return narrow ? batch_kernel<1, uint32_t, int32_t> : batch_kernel<1, uint64_t, int32_t>;
        case 2: return narrow ? batch_kernel<2, uint32_t, int32_t> : batch_kernel<2, uint64_t, int32_t>;
        case 4: return batch_kernel<4, uint64_t, int32_t>;
        default: return batch_kernel<kMaxExpPoly, uint64_t, int32_t>;
    }
}

int launch_batch(const BatchArgs &b, const BatchLaunch &bl, void *stream, std::string &err) {
    BatchKernelFn fn = bl.z16 ? batch_kernel_z16(bl.maxe_class, bl.narrow) : batch_kernel_z32(bl.maxe_class, bl.narrow);
    const int lds = b.lds_words * (int)sizeof(int32_t);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) {
            err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    // dense teams and lane kernels first, beside the persistent kernel where a side stream is given
    const bool teams = (!bl.teams.empty() || !bl.lanes.empty()) && b.sweep_limit == 0;
    if (teams) {
        void *s = bl.side_stream ? bl.side_stream : stream;
        hipError_t e = hipSuccess;
        if (bl.side_stream) {
            e = hipEventRecord((hipEvent_t)bl.fork, (hipStream_t)stream);
            if (e == hipSuccess) e = hipStreamWaitEvent((hipStream_t)s, (hipEvent_t)bl.fork, 0);
        }
        for (const TeamGroup &g : bl.teams) {
            if (e != hipSuccess) break;
            int rc = launch_team_group(b.insts, bl.settled_tasks, g, s, err);
            if (rc != SA_OK) return rc;
        }
        for (const LaneGroup &g : bl.lanes) {
            if (e != hipSuccess) break;
            int rc = launch_lane_group(bl.lane_args, bl.settled_tasks, g, s, err);
            if (rc != SA_OK) return rc;
        }
        if (bl.side_stream && e == hipSuccess) e = hipEventRecord((hipEvent_t)bl.join, (hipStream_t)s);
        if (e != hipSuccess) {
            err = std::string("batch launch: ") + hipGetErrorString(e);
            return SA_EDEVICE;
        }
    }
    auto join = [&]() -> int {
        if (!teams || !bl.side_stream) return SA_OK;
        hipError_t e = hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)bl.join, 0);
        if (e == hipSuccess) return SA_OK;
        err = std::string("batch launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    };
    if (b.n_tasks == 0) return join();
    int32_t n_settled = 0;
    for (const SettledGroup &g : bl.settled) n_settled += g.n;
    BatchArgs a = b;
    auto persistent = [&](int32_t phase) {
        a.phase = phase;
        hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, a.counter);
        hipLaunchKernelGGL(fn, dim3((unsigned)bl.groups), dim3((unsigned)(kBatchWaves * kWave)), (size_t)lds,
                           (hipStream_t)stream, a);
    };
    if (n_settled == 0 || b.sweep_limit > 0) {
        persistent(kPhaseWhole);
    } else {
        persistent(kPhaseFirst);
        for (const SettledGroup &g : bl.settled) {
            if (g.n == 0) continue;
            int rc = launch_settled_batch(b.insts, bl.settled_tasks + g.first, g.n, g.lds_bytes, bl.maxe_class, stream, err);
            if (rc != SA_OK) return rc;
        }
        persistent(kPhaseLast);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("batch launch: ") + hipGetErrorString(e);
        return SA_EDEVICE;
    }
    return join();
}

}  // namespace sa
