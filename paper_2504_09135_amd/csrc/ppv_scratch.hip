// Scratch areas in which the workgroups that share a row meet (see SplitRow): work that may run at the same time never shares one.
// Eager calls: one area per (device, stream), so that calls on different streams never share one; allocated at the first call
// that needs it.  hipStreamPerThread is one handle for as many streams as there are threads: such a stream is known by its
// thread's number (never used again after the thread), and the first MOST_THREADS of them have an area.
// Captured calls: one area per (device, capture, stream of it), since a graph may be replayed anywhere, beside another graph and
// beside eager calls on the stream it came from.  Nothing can be allocated during a capture: SPARES areas lie ready on a device
// from the first eager call on that splits rows there, and later eager calls make up for those that were taken, up to MOST_CAPTURED.
// A capture that finds none, or more rows than such an area has, does not split rows.
// How long a graph lives is not known here: every area is kept until the process ends.
#include <atomic>
#include <cstddef>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "ppv_internal.h"

namespace {
constexpr uint64_t MOST_THREADS = 64;
constexpr int SPARES = 4, MOST_CAPTURED = 256;   // 1.9 MB each
constexpr int CAPTURED_ROWS = 128;               // twice as many rows as workgroups for them are not split

std::mutex g_mu;
std::map<std::tuple<int, hipStream_t, uint64_t, unsigned long long>, SplitScratch *> g_areas;   // device, stream, thread's number or 0, capture's or 0
struct Device {
    std::vector<SplitScratch *> spare;   // zeroed
    int made = 0;                        // spare and taken
    bool failed = false;                 // the last one could not be had: not tried again
};
std::map<int, Device> g_device;

uint64_t thread_number() {   // 1, 2, ...
    static std::atomic<uint64_t> last{0};
    thread_local const uint64_t mine = ++last;
    return mine;
}
size_t bytes_for(int rows) { return offsetof(SplitScratch, row) + (size_t)rows * sizeof(SplitRow); }
SplitScratch *new_area(int rows) {
    const size_t bytes = bytes_for(rows);
    SplitScratch *p = nullptr;
    hipError_t e = hipMalloc((void **)&p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        ppv_pool_empty();
        e = hipMalloc((void **)&p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}
// Areas for captures to come.  They are zeroed on a stream of their own and waited for: what is replayed first, and
// where, is not known.  (Another thread may be capturing: with the capture mode relaxed that does not forbid these calls.)
void lay_ready(Device &d) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    hipStream_t own = nullptr;
    bool ok = relaxed && hipStreamCreateWithFlags(&own, hipStreamNonBlocking) == hipSuccess;
    std::vector<SplitScratch *> made;
    while (ok && (int)(d.spare.size() + made.size()) < SPARES && d.made + (int)made.size() < MOST_CAPTURED) {
        SplitScratch *p = new_area(CAPTURED_ROWS);
        ok = p && hipMemsetAsync(p, 0, bytes_for(CAPTURED_ROWS), own) == hipSuccess;
        if (p) made.push_back(p);
    }
    if (own) {
        const bool waited = hipStreamSynchronize(own) == hipSuccess;
        (void)hipStreamDestroy(own);
        if (ok && waited) {
            d.spare.insert(d.spare.end(), made.begin(), made.end());
            d.made += (int)made.size();
            made.clear();
        }
    }
    for (SplitScratch *p : made) (void)hipFree(p);
    d.failed = !made.empty() || !ok;
    (void)hipGetLastError();
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
}
SplitScratch *area_for(hipStream_t stream, int rows) {
    int dev = 0;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    unsigned long long capture = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    // (no answer: the legacy stream while another one is captured, on which nothing can be allocated)
    const bool known = hipStreamGetCaptureInfo(stream, &cs, &capture) == hipSuccess;
    if (!known) (void)hipGetLastError();
    const bool captured = known && cs != hipStreamCaptureStatusNone;
    const uint64_t thread = stream == hipStreamPerThread ? thread_number() : 0;
    if (thread > MOST_THREADS || (captured && (cs != hipStreamCaptureStatusActive || rows > CAPTURED_ROWS))) return nullptr;
    std::lock_guard<std::mutex> lock(g_mu);
    Device &d = g_device[dev];
    const auto key = std::make_tuple(dev, stream, thread, captured ? capture : 0ull);
    const auto it = g_areas.find(key);
    SplitScratch *p = it != g_areas.end() ? it->second : nullptr;
    if (captured) {
        if (p || d.spare.empty()) return p;
        p = d.spare.back();
        g_areas[key] = p;
        d.spare.pop_back();
        return p;
    }
    if (!known) return p;
    if (!p) {
        p = new_area(PPV_SPLIT_MAX_ROWS);
        if (!p) return nullptr;
        // an area starts as zeros, which no call has for a mark; in stream order before the kernel that is about to be launched
        if (hipMemsetAsync(p, 0, bytes_for(PPV_SPLIT_MAX_ROWS), stream) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipFree(p);
            return nullptr;
        }
        g_areas[key] = p;
    }
    if ((int)d.spare.size() < SPARES && d.made < MOST_CAPTURED && !d.failed) lay_ready(d);
    return p;
}
}  // namespace

SplitScratch *ppv_split_scratch(hipStream_t stream, int rows) {
    try {
        return area_for(stream, rows);
    } catch (...) {   // (no memory for the tables above)
        return nullptr;
    }
}
