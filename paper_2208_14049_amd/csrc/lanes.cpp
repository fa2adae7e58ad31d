// The process-wide set of streams that handles issue their kernels on (see LANES in engine.h).
#include <mutex>

#include "engine.h"

namespace ens {

namespace {
constexpr int MAX_DEVICES = 64;
struct LaneSet {
    int users = 0;
    int first = 0;                 // of the next handle: those with work for one lane do not all meet on the same one
    hipStream_t s[LANES] = {nullptr, nullptr, nullptr, nullptr};
};
std::mutex g_lock;
LaneSet g_sets[MAX_DEVICES];

void destroy(LaneSet& set) {
    for (hipStream_t& s : set.s) {
        if (s) (void)hipStreamDestroy(s);
        s = nullptr;
    }
}
}  // namespace

hipError_t acquire_lanes(hipStream_t* lanes) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> hold(g_lock);
    LaneSet& set = g_sets[dev];
    if (set.users == 0) {
        int units = 0;
        e = hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        std::vector<uint32_t> every((size_t)(units + 31) / 32, 0xFFFFFFFFu);
        if (units % 32) every.back() = (1u << (units % 32)) - 1u;
        for (hipStream_t& s : set.s) {
            e = hipExtStreamCreateWithCUMask(&s, (uint32_t)every.size(), every.data());
            if (e != hipSuccess) {
                destroy(set);
                return e;
            }
        }
    }
    set.users++;
    for (int i = 0; i < LANES; i++) lanes[i] = set.s[(set.first + i) % LANES];
    set.first = (set.first + 1) % LANES;
    return hipSuccess;
}

void release_lanes(const hipStream_t* lanes) {
    std::lock_guard<std::mutex> hold(g_lock);
    for (LaneSet& set : g_sets)
        for (const hipStream_t s : set.s)
            if (set.users > 0 && s == lanes[0]) {
                if (--set.users == 0) destroy(set);
                return;
            }
}

}  // namespace ens
