// Linked against libsa.so with a hipMalloc that finds no room: the lane image and the order list are
// speed-ups, and a run goes on without them. Prints "ok".
#include <cstdio>
#include <string>
#include <vector>

#include "../paper_2511_17245_amd/csrc/sa_plan.h"

static int asked = 0;
extern "C" hipError_t hipMalloc(void **p, size_t) {
    ++asked;
    *p = nullptr;
    return hipErrorOutOfMemory;
}
extern "C" hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t attr, int) {
    if (attr == hipDeviceAttributeMultiprocessorCount) *value = 256;
    else if (attr == hipDeviceAttributeMaxSharedMemoryPerBlock) *value = 160 * 1024;
    else return hipErrorInvalidValue;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipFree(void *) { return hipSuccess; }

int main() {
    // a ring of 600 variables with chords: a problem the lane kernel takes
    const int n = 600;
    std::vector<int64_t> ptr{0}, coef;
    std::vector<int32_t> fac, lo((size_t)n, -5), hi((size_t)n, 5);
    for (int i = 0; i < n; ++i)
        for (int d : {7, 60}) {
            fac.push_back(i);
            fac.push_back((i * 31 + d) % n == i ? (i + 1) % n : (i * 31 + d) % n);
            ptr.push_back((int64_t)fac.size());
            coef.push_back(1 + i % 5);
        }
    sa_instance in{n, (int64_t)coef.size(), ptr.data(), fac.data(), coef.data()};
    sa_bounds bd{lo.data(), hi.data()};
    sa::Canonical c;
    std::string err;
    sa_plan plan;
    plan.rule = SA_HEAT_BATH;
    if (sa::canonicalize(&in, &bd, c, err) != SA_OK || sa::pack(c, plan.packed, err) != SA_OK) return 2;
    plan.dp.n = n;
    plan.dp.coef32 = 1;
    sa::LaneChoice lane;
    sa::LaneArgs args{};
    int bad = 0;
    if (sa::choose_lane_run(&plan, 4, 100, lane, args) != SA_OK || lane.waves != 0) bad |= 1;
    const int lanes_asked = asked;
    if (lanes_asked == 0) bad |= 2;   // (the problem is one the lane kernel takes)
    sa_plan::Sched *order = &plan.order;
    if (sa::get_order_if_room(&plan, &order) != SA_OK || order != nullptr) bad |= 4;
    if (asked == lanes_asked) bad |= 8;
    if (bad) {
        std::fprintf(stderr, "FAILED: %d\n", bad);
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
