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

int SideStream::create() {
    hipError_t e = hipStreamCreateWithFlags((hipStream_t *)&stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags((hipEvent_t *)&fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags((hipEvent_t *)&join, hipEventDisableTiming);
    return (int)e;
}

void SideStream::destroy() {
    if (fork) (void)hipEventDestroy((hipEvent_t)fork);
    if (join) (void)hipEventDestroy((hipEvent_t)join);
    if (stream) (void)hipStreamDestroy((hipStream_t)stream);
    stream = fork = join = nullptr;
}

int SideStream::fork_from(void *main) const {
    hipError_t e = hipEventRecord((hipEvent_t)fork, (hipStream_t)main);
    if (e == hipSuccess) e = hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)fork, 0);
    return (int)e;
}

int SideStream::mark() const { return (int)hipEventRecord((hipEvent_t)join, (hipStream_t)stream); }

int SideStream::join_to(void *main) const { return (int)hipStreamWaitEvent((hipStream_t)main, (hipEvent_t)join, 0); }

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
    // `stream` waits for every side stream that was forked from it, also where a launch fails: the caller, who
    // knows of `stream` alone, gives the buffers back after it.
    const SideStream *open[2] = {nullptr, nullptr};
    auto join = [&]() -> int {
        int first = 0;
        for (const SideStream *&side : open) {
            if (!side) continue;
            int e = side->mark();
            if (!e) e = side->join_to(stream);
            if (!first) first = e;
            side = nullptr;
        }
        return first;
    };
    auto failed = [&](int e) {
        err = std::string("batch launch: ") + hipGetErrorString((hipError_t)e);
        (void)join();
        return SA_EDEVICE;
    };
    // dense teams and lane kernels first, beside the persistent kernel where a side stream is given
    const bool teams = (!bl.teams.empty() || !bl.lanes.empty()) && b.sweep_limit == 0;
    const bool beside = teams && bl.beside.stream;
    if (teams) {
        void *s = beside ? bl.beside.stream : stream;
        if (beside) {
            open[0] = &bl.beside;
            if (int e = bl.beside.fork_from(stream)) return failed(e);
        }
        int rc = SA_OK;
        for (size_t i = 0; rc == SA_OK && i < bl.teams.size(); ++i)
            rc = launch_team_group(b.insts, bl.settled_tasks, bl.teams[i], s, err);
        for (size_t i = 0; rc == SA_OK && i < bl.lanes.size(); ++i)
            rc = launch_lane_group(bl.lane_args, bl.settled_tasks, bl.lanes[i], s, err);
        if (rc != SA_OK) {
            (void)join();
            return rc;
        }
    }
    if (b.n_tasks == 0) {
        const int e = join();
        return e ? failed(e) : SA_OK;
    }
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
        // A group's end runs on few replicas: the groups beside each other, the largest (the first there
        // is) on the batch's stream, the others in their order on the side stream (64 mixed problems:
        // 14.1, 8.4 and 7.5 ms of settled kernels in a row before, the run 113 -> 103 ms).
        void *s = stream;
        bool forked = false;
        int left = 0;
        for (const SettledGroup &g : bl.settled) left += g.n > 0;
        for (const SettledGroup &g : bl.settled) {
            if (g.n == 0) continue;
            if (s == stream && --left > 0 && bl.settled_side.stream) {
                open[1] = &bl.settled_side;
                if (int e = bl.settled_side.fork_from(stream)) return failed(e);
                forked = true;
            }
            int rc = launch_settled_batch(b.insts, bl.settled_tasks + g.first, g.n, g.lds_bytes, bl.maxe_class, s, err);
            if (rc != SA_OK) {
                (void)join();
                return rc;
            }
            if (forked) s = bl.settled_side.stream;
        }
        if (forked) {
            int e = bl.settled_side.mark();
            if (!e) e = bl.settled_side.join_to(stream);
            if (e) return failed(e);
            open[1] = nullptr;
        }
        persistent(kPhaseLast);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return failed(e);
    const int je = join();
    return je ? failed(je) : SA_OK;
}

}  // namespace sa
