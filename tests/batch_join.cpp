// Linked against libsa.so with launches, events and waits that are only written down: after launch_batch, also
// when its n-th launch fails, the caller's stream waits for everything queued on the side streams. Prints "ok".
#include <cstdio>
#include <map>
#include <string>
#include <vector>

#include "../paper_2511_17245_amd/csrc/sa_internal.h"
#include <hip/hip_runtime_api.h>

namespace {
std::map<void *, int> queued, seen_by_main;   // launches on a stream; those that the main stream waits for
std::map<void *, std::pair<void *, int>> recorded;   // event: stream and its launches then
void *const kMain = (void *)0x100;
int launches, fail_at;
hipError_t last = hipSuccess;
void *config_stream;
}  // namespace

extern "C" {
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t s) {
    config_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
    *g = *b = dim3(1, 1, 1);
    *m = 0;
    *s = (hipStream_t)config_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s) {
    if (++launches == fail_at) return last = hipErrorLaunchFailure;
    ++queued[s];
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    recorded[e] = {s, queued[s]};
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (s == kMain) seen_by_main[recorded[e].first] = recorded[e].second;
    return hipSuccess;
}
}

int main() {
    sa::BatchArgs a{};
    a.n_tasks = 1;
    a.lds_words = 64;
    sa::BatchLaunch bl;
    bl.beside.stream = (void *)0x200;
    bl.beside.fork = (void *)0x201;
    bl.beside.join = (void *)0x202;
    bl.settled_side.stream = (void *)0x300;
    bl.settled_side.fork = (void *)0x301;
    bl.settled_side.join = (void *)0x302;
    for (int i = 0; i < 2; ++i) {
        sa::TeamGroup t;
        t.n = 1;
        t.waves = 4;
        t.rule = SA_METROPOLIS;
        t.small = true;
        bl.teams.push_back(t);
        sa::LaneGroup l;
        l.n = 1;
        l.waves = 1;
        bl.lanes.push_back(l);
    }
    for (sa::SettledGroup &g : bl.settled) g.n = 1;
    int total = 0, bad = 0;
    for (int tasks = 1; tasks >= 0; --tasks) {
        a.n_tasks = tasks;
        for (fail_at = 0;; ++fail_at) {
            queued.clear();
            seen_by_main.clear();
            recorded.clear();
            launches = 0;
            last = hipSuccess;
            std::string err;
            const int rc = sa::launch_batch(a, bl, kMain, err);
            if (fail_at == 0) total = launches;
            if ((rc != SA_OK) != (fail_at > 0)) {
                std::fprintf(stderr, "FAILED: %d tasks, launch %d of %d fails, returns %d\n", tasks, fail_at, total, rc);
                ++bad;
            }
            for (void *side : {bl.beside.stream, bl.settled_side.stream})
                if (seen_by_main[side] != queued[side]) {
                    std::fprintf(stderr, "FAILED: %d tasks, launch %d of %d fails: %d launches on %p, %d waited for\n", tasks, fail_at,
                                 total, queued[side], side, seen_by_main[side]);
                    ++bad;
                }
            if (fail_at == 0 && total < (tasks ? 11 : 4)) ++bad;   // 2 teams, 2 lanes; 2 x (reset, persistent), 3 settled
            if (fail_at == total) break;
        }
    }
    if (bad) return 1;
    std::printf("ok\n");
    return 0;
}
