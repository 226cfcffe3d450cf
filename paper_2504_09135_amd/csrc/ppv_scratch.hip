// Scratch areas in which the workgroups that share a row meet (see SplitRow).  One per (device, stream), so that
// calls on different streams never share one; allocated at the first call that needs it and kept until the
// process ends.  A stream that is being captured cannot allocate: it gets an area only if it already has one.
// hipStreamPerThread is one handle for as many streams as there are threads: such a stream is known by its thread's number
// (never used again after the thread), and the first MOST_THREADS of them have an area.
#include <atomic>
#include <map>
#include <mutex>
#include <tuple>

#include "ppv_internal.h"

namespace {
std::mutex g_mu;
std::map<std::tuple<int, hipStream_t, uint64_t>, SplitScratch *> g_scratch;
constexpr uint64_t MOST_THREADS = 64;
uint64_t thread_number() {   // 1, 2, ...
    static std::atomic<uint64_t> last{0};
    thread_local const uint64_t mine = ++last;
    return mine;
}
bool captured(hipStream_t stream) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone) return false;
    (void)hipGetLastError();
    return true;
}
}  // namespace

SplitScratch *ppv_split_scratch(hipStream_t stream, bool eager_only) {
    if (eager_only && captured(stream)) return nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_mu);
    const uint64_t thread = stream == hipStreamPerThread ? thread_number() : 0;
    if (thread > MOST_THREADS) return nullptr;
    const auto key = std::make_tuple(dev, stream, thread);
    const auto it = g_scratch.find(key);
    if (it != g_scratch.end()) return it->second;
    if (captured(stream)) return nullptr;
    SplitScratch *p = nullptr;
    hipError_t e = hipMalloc((void **)&p, sizeof(SplitScratch));
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        ppv_pool_empty();
        e = hipMalloc((void **)&p, sizeof(SplitScratch));
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    // the arrival counters start at zero (afterwards every launch leaves them at zero); in stream order before the
    // kernel that is about to be launched
    if (hipMemsetAsync(p->arrivals, 0, sizeof(p->arrivals), stream) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(p);
        return nullptr;
    }
    g_scratch[key] = p;
    return p;
}
