// Memory of the index builder that is worth keeping from one build to the next, and the upload of a constraint set.
//
// What bounds it: building the index of 1M sequences (18M tokens, 0.6 GB of arrays) takes the GPU under a millisecond,
// but mapping and unmapping that memory (34 hipMalloc, 27 hipFree) took 6 ms of a 16 ms build, and the driver's copy
// from pageable memory another 2.6 ms (31 GB/s; 57 from pinned memory).
//
// Device blocks: ppv_pool_take hands out a block of at least the size asked for, from the blocks that were given back
// or from hipMalloc; ppv_pool_give keeps it for the next taker.  At most POOL_KEEP bytes are kept per process, for at
// most POOL_AGE from their last use, and all of them go back to the system when an allocation of this library fails.
// Whoever gives a block back has waited for the device to be done with it; a block whose wait failed goes to hipFree, which
// waits by itself.  The pinned memory of the upload goes back after the same time.
// The age is looked at by a thread that is there while anything is kept: a process that makes no further call would
// otherwise hold the memory until it ends.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <mutex>
#include <new>
#include <thread>
#include <unordered_map>
#include <vector>

#include <sched.h>
#include <unistd.h>

#include "ppv_internal.h"

#ifndef PPV_POOL_AGE_MS   // (a test builds this file with less)
#define PPV_POOL_AGE_MS 20000
#endif

namespace {

using Clock = std::chrono::steady_clock;
constexpr size_t POOL_KEEP = 1ull << 30;
constexpr std::chrono::milliseconds POOL_AGE(PPV_POOL_AGE_MS);
constexpr size_t POOL_ROUND = 256u << 10;

// What is freed here is in nobody's use, so freeing it is no part of a capture that some stream may be in.
struct OutsideCaptures {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    OutsideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~OutsideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};
bool free_block(void *p) {
    const OutsideCaptures outside;
    if (hipFree(p) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

struct Kept {
    void *p;
    size_t bytes;
    int device;
    bool leaving;               // the watching thread is freeing it
    Clock::time_point since;
};
struct Pool {
    std::mutex mu;
    std::condition_variable cv;
    std::vector<Kept> kept;                                        // oldest first
    std::unordered_map<void *, std::pair<size_t, int>> out;        // blocks in use: size, device
    size_t kept_bytes = 0;
    std::thread watch;
    pid_t pid = 0;              // the process `watch` belongs to (a forked child has no such thread)
    bool watching = false, ending = false;
    bool more = false;          // something has been kept since `watch` last looked

    void erase(size_t i) {
        kept_bytes -= kept[i].bytes;
        kept.erase(kept.begin() + (long)i);
    }
    // frees kept blocks, oldest first, until at most `most` bytes are kept; one that cannot be freed stays on the list
    void shrink(size_t most) {
        for (size_t i = 0; i < kept.size() && kept_bytes > most;)
            if (!kept[i].leaving && free_block(kept[i].p)) erase(i);
            else i++;
    }
};
Pool &pool() {
    static Pool *p = new Pool;   // never destroyed: the HIP runtime may be gone before a static's destructor runs
    return *p;
}

bool give_back_ring(Clock::time_point now, Clock::time_point *next);   // the upload's pinned memory, below

void watch_kept() {
    Pool &p = pool();
    std::unique_lock<std::mutex> lock(p.mu);
    while (!p.ending) {
        p.more = false;
        const Clock::time_point now = Clock::now();
        Clock::time_point next = now + POOL_AGE;
        lock.unlock();
        const bool ring = give_back_ring(now, &next);
        lock.lock();
        bool any = false;
        for (size_t i = 0; i < p.kept.size() && !p.ending;) {
            any = true;
            if (p.kept[i].since + POOL_AGE > now) {
                next = std::min(next, p.kept[i].since + POOL_AGE);
                break;   // (the others are younger)
            }
            void *const q = p.kept[i].p;
            p.kept[i].leaving = true;
            lock.unlock();   // (hipFree waits for the device: nobody else has to)
            const bool gone = free_block(q);
            lock.lock();
            i = 0;
            while (p.kept[i].p != q) i++;   // (only this thread erases a block that is leaving)
            if (gone) {
                p.erase(i);
            } else {   // another time
                Kept k = p.kept[i];
                k.leaving = false;
                k.since = Clock::now();
                p.kept.erase(p.kept.begin() + (long)i);
                p.kept.push_back(k);
            }
            i = 0;
        }
        if (!any && !ring) {
            if (!p.more) break;
        } else if (!p.ending) {
            p.cv.wait_until(lock, next);
        }
    }
    p.watching = false;
}
// At the process's end, before the HIP runtime goes (which was there first).
void stop_watching() {
    Pool &p = pool();
    if (p.pid != getpid()) return;
    {
        std::lock_guard<std::mutex> lock(p.mu);
        p.ending = true;
        p.cv.notify_all();
    }
    if (p.watch.joinable()) p.watch.join();
}
// sees to it that the thread is there; with p.mu held
bool see_to_watch(Pool &p) {
    p.more = true;
    if (p.watching && p.pid == getpid()) return true;
    if (p.ending) return true;   // the process is about to end
    try {
        if (p.pid == 0 && atexit(stop_watching) != 0) return false;
        if (p.watch.joinable()) {
            if (p.pid == getpid()) p.watch.join();   // (it has left its loop: nothing was kept)
            else p.watch.detach();
        }
        p.pid = getpid();
        p.watch = std::thread(watch_kept);
        p.watching = true;
        return true;
    } catch (...) {
        return false;
    }
}

}  // namespace

ppv_status ppv_pool_take(void **out, size_t bytes, size_t *got) {
    *out = nullptr;
    int dev = 0;
    PPV_HIP_TRY(hipGetDevice(&dev));
    const size_t need = (std::max<size_t>(bytes, 1) + POOL_ROUND - 1) / POOL_ROUND * POOL_ROUND;
    Pool &p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    try {
        p.out.reserve(p.out.size() + 1);
        p.kept.reserve(p.kept.size() + p.out.size() + 1);   // so that giving a block back cannot fail
        size_t best = p.kept.size();
        for (size_t i = 0; i < p.kept.size(); i++)   // the smallest that fits and is not much too large
            if (!p.kept[i].leaving && p.kept[i].device == dev && p.kept[i].bytes >= need && p.kept[i].bytes <= need + need / 2 &&
                (best == p.kept.size() || p.kept[i].bytes < p.kept[best].bytes))
                best = i;
        if (best < p.kept.size()) {
            const Kept k = p.kept[best];
            p.out[k.p] = {k.bytes, k.device};
            p.erase(best);
            *out = k.p;
            if (got) *got = k.bytes;
            return PPV_OK;
        }
        void *q = nullptr;
        hipError_t e = hipMalloc(&q, need);
        if (e == hipErrorOutOfMemory && !p.kept.empty()) {
            (void)hipGetLastError();
            p.shrink(0);
            e = hipMalloc(&q, need);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e == hipErrorOutOfMemory ? PPV_ENOMEM : PPV_EDEVICE;
        }
        p.out[q] = {need, dev};
        *out = q;
        if (got) *got = need;
        return PPV_OK;
    } catch (const std::bad_alloc &) {
        return PPV_ENOMEM;
    }
}

void ppv_pool_give(void *q, bool over) {
    if (!q) return;
    Pool &p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    const auto it = p.out.find(q);
    if (it == p.out.end()) return;
    const size_t bytes = it->second.first;
    const int dev = it->second.second;
    p.out.erase(it);
    if (bytes > POOL_KEEP || !over || !see_to_watch(p)) {
        (void)free_block(q);
        return;
    }
    p.kept.push_back({q, bytes, dev, false, Clock::now()});
    p.kept_bytes += bytes;
    p.shrink(POOL_KEEP);
}

void ppv_pool_empty() {
    Pool &p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    p.shrink(0);
}

// ------------------------------------------------------------------------------------------
// A few words of pinned memory that a kernel writes and the host reads after one synchronisation (a copy back to
// pageable memory is two more trips).
namespace {
constexpr int WORD_SLOTS = 64;
std::mutex g_words_mu;
std::condition_variable g_words_cv;
unsigned char *g_words;      // WORD_SLOTS slots of PPV_HOST_WORDS_BYTES (4 KB), kept until the process ends
uint64_t g_words_taken;
}  // namespace

void *ppv_host_words_take() {
    std::unique_lock<std::mutex> lock(g_words_mu);
    if (!g_words && hipHostMalloc((void **)&g_words, WORD_SLOTS * PPV_HOST_WORDS_BYTES, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
        g_words = nullptr;
        return nullptr;
    }
    // (as many builds at a time as there are slots; the next one waits for any of them to end, which needs no slot)
    while (g_words_taken == ~0ull) g_words_cv.wait(lock);
    const int i = __builtin_ctzll(~g_words_taken);
    g_words_taken |= 1ull << i;
    return g_words + (size_t)i * PPV_HOST_WORDS_BYTES;
}
void ppv_host_words_give(void *p) {
    if (!p) return;
    std::lock_guard<std::mutex> lock(g_words_mu);
    g_words_taken &= ~(1ull << (((unsigned char *)p - g_words) / PPV_HOST_WORDS_BYTES));
    g_words_cv.notify_one();
}

// ------------------------------------------------------------------------------------------
// Upload.  Tokens travel as 16-bit words (and a plane of upper bytes where the vocabulary needs one), offsets as
// 32-bit words, through a ring of pinned slots: a few threads check and pack, the calling thread hands finished slots to
// the copy engine in order, several neighbours per copy.  (40 MB in copies of 0.5 / 1 / 2 / 4 MB: 28 / 38 / 46 / 50 GB/s;
// packing: 28 GB/s of input with one thread, 97 with four, 123 with eight.)
namespace {

constexpr int UP_THREADS = 8;                  // at most
constexpr size_t UP_TOKENS = 256u << 10;       // tokens per slot
constexpr size_t UP_OFFSETS = UP_TOKENS / 2;   // offsets per slot
constexpr size_t UP_LO = UP_TOKENS * 2;        // bytes of a slot in the ring of 16-bit words (or offsets) ...
constexpr size_t UP_HI = UP_TOKENS;            // ... and in the ring of upper bytes
constexpr size_t UP_SLOTS = 64;
constexpr size_t UP_RUN = 4, UP_RUN_MOST = 16; // slots per copy: at least (but for the last), at most
struct Stage {
    std::mutex mu;                             // one upload at a time: the bus is the bottleneck
    unsigned char *buf = nullptr;              // the two rings (48 MB), pinned, kept for POOL_AGE after an upload; where
    bool pinned = false;                       // no pinned memory is to be had, ordinary memory, which the runtime stages
    Clock::time_point since;                   // the end of the last upload
    hipEvent_t ev[UP_SLOTS] = {};              // the end of the copy whose last slot this is
    int copy_of[UP_SLOTS];                     // the slot that the copy of this slot ended with; -1: none under way
    int device = -1;                           // the device the events belong to

    bool wait(size_t k) {                      // until slot k may be filled; it may hold a copy of the upload before
        const int e = copy_of[k];
        if (e < 0) return true;
        if (hipEventSynchronize(ev[e]) != hipSuccess) return false;
        for (int &c : copy_of)
            if (c == e) c = -1;
        return true;
    }
    ppv_status ready(int dev) {
        if (!buf) {
            for (int &c : copy_of) c = -1;
            pinned = hipHostMalloc((void **)&buf, UP_SLOTS * (UP_LO + UP_HI), hipHostMallocPortable) == hipSuccess;
            if (!pinned) {
                (void)hipGetLastError();
                buf = (unsigned char *)malloc(UP_SLOTS * (UP_LO + UP_HI));
            }
            if (!buf) return PPV_ENOMEM;
        }
        if (device == dev) return PPV_OK;
        for (size_t i = 0; i < UP_SLOTS; i++)
            if (!wait(i)) return PPV_EDEVICE;
        drop_events();
        for (hipEvent_t &e : ev) PPV_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        device = dev;
        return PPV_OK;
    }
    void drop_events() {
        for (hipEvent_t &e : ev) {
            if (e) (void)hipEventDestroy(e);
            e = nullptr;
        }
        device = -1;
    }
    void drop() {   // (a copy that may still read the buffer: it stays)
        if (!buf) return;
        const OutsideCaptures outside;
        for (size_t i = 0; i < UP_SLOTS; i++)
            if (!wait(i)) return;
        drop_events();
        if (!pinned) free(buf);
        else if (hipHostFree(buf) != hipSuccess) (void)hipGetLastError();
        buf = nullptr;
    }
};
Stage &stage() {
    static Stage *s = new Stage;
    return *s;
}

// Gives the ring back if the last upload is POOL_AGE ago; else lowers *next to when that will be.  Whether there is a ring.
bool give_back_ring(Clock::time_point now, Clock::time_point *next) {
    Stage &sg = stage();
    const std::unique_lock<std::mutex> lock(sg.mu, std::try_to_lock);
    if (!lock.owns_lock()) return true;   // in use: look again after POOL_AGE
    if (sg.buf && sg.since + POOL_AGE <= now) sg.drop();
    if (sg.buf && sg.since + POOL_AGE > now) *next = std::min(*next, sg.since + POOL_AGE);
    return sg.buf != nullptr;
}

int cpus() {
    cpu_set_t set;
    const int n = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) : 1;
    return n > 1 ? n : 1;
}

// One job: a slot's worth of offsets (the first off_jobs) or of tokens.
struct Upload {
    const int32_t *tokens;
    const int64_t *offsets;
    size_t total, n_off, off_jobs, jobs;
    uint32_t vocab;
    bool wide;
    std::atomic<bool> invalid{false};
    std::atomic<int64_t> longest{0};

    void pack(size_t job, unsigned char *buf, uint8_t *hi) {
        if (job < off_jobs) {   // offsets first: they say whether the set is well formed
            const size_t a = job * UP_OFFSETS, n = std::min(UP_OFFSETS, n_off - a);
            uint32_t *o = (uint32_t *)buf;
            const int64_t *in = offsets + a;
            int64_t before = a ? offsets[a - 1] : -1, least = 1, most = 0;
            for (size_t i = 0; i < n; i++) {
                const int64_t len = in[i] - before;
                before = in[i];
                o[i] = (uint32_t)in[i];
                least = std::min(least, len);
                if (a + i > 0) most = std::max(most, len);
            }
            if (least < 1) invalid = true;
            int64_t cur = longest.load();
            while (cur < most && !longest.compare_exchange_weak(cur, most)) {
            }
        } else {
            const size_t a = (job - off_jobs) * UP_TOKENS, n = std::min(UP_TOKENS, total - a);
            uint16_t *lo = (uint16_t *)buf;
            const uint32_t *in = (const uint32_t *)tokens + a;
            uint32_t bad = 0;
            if (!wide) {
                for (size_t i = 0; i < n; i++) {
                    bad |= (uint32_t)(in[i] >= vocab);
                    lo[i] = (uint16_t)in[i];
                }
            } else {
                for (size_t i = 0; i < n; i++) {
                    bad |= (uint32_t)(in[i] >= vocab);
                    lo[i] = (uint16_t)in[i];
                    hi[i] = (uint8_t)(in[i] >> 16);
                }
            }
            if (bad) invalid = true;
        }
    }
    // jobs job .. job + n - 1, all of one kind, from neighbouring slots
    hipError_t copy(size_t job, size_t n, const unsigned char *buf, const uint8_t *hi, uint16_t *d_lo, uint8_t *d_hi,
                    uint32_t *d_off, hipStream_t st) const {
        if (job < off_jobs) {
            const size_t a = job * UP_OFFSETS, m = std::min(n * UP_OFFSETS, n_off - a);
            return hipMemcpyAsync(d_off + a, buf, m * sizeof(uint32_t), hipMemcpyHostToDevice, st);
        }
        const size_t a = (job - off_jobs) * UP_TOKENS, m = std::min(n * UP_TOKENS, total - a);
        const hipError_t e = hipMemcpyAsync(d_lo + a, buf, m * sizeof(uint16_t), hipMemcpyHostToDevice, st);
        if (!wide || e != hipSuccess) return e;
        return hipMemcpyAsync(d_hi + a, hi, m, hipMemcpyHostToDevice, st);
    }
};

}  // namespace

ppv_status ppv_upload_set(const int32_t *tokens, const int64_t *offsets, int64_t n_seq, int32_t vocab, uint16_t *d_lo,
                          uint8_t *d_hi, uint32_t *d_off, hipStream_t st, int32_t *l_max) {
    Upload up;
    up.tokens = tokens;
    up.offsets = offsets;
    up.total = (size_t)offsets[n_seq];
    up.n_off = (size_t)n_seq + 1;
    up.vocab = (uint32_t)vocab;
    up.wide = d_hi != nullptr;
    up.off_jobs = (up.n_off + UP_OFFSETS - 1) / UP_OFFSETS;
    up.jobs = up.off_jobs + (up.total + UP_TOKENS - 1) / UP_TOKENS;
    int dev = 0;
    PPV_HIP_TRY(hipGetDevice(&dev));
    Stage &sg = stage();
    std::lock_guard<std::mutex> lock(sg.mu);
    struct Used {   // whatever comes of it: the ring's time starts again
        Stage &sg;
        ~Used() {
            sg.since = Clock::now();
            Pool &p = pool();
            std::lock_guard<std::mutex> plock(p.mu);
            if (!see_to_watch(p)) sg.drop();
        }
    } used{sg};
    const ppv_status ready = sg.ready(dev);
    if (ready != PPV_OK) return ready;
    bool failed = false;

    unsigned char *lo = sg.buf;
    uint8_t *hi = sg.buf + UP_SLOTS * UP_LO;

    const int threads = up.jobs < 4 ? 0 : (int)std::min<size_t>(std::min(UP_THREADS, cpus() - 1), up.jobs);
    // job j uses slot j % UP_SLOTS; `open`: jobs whose slot is free; packed[k]: how many jobs slot k has held
    std::atomic<size_t> next{0}, open{0};
    std::atomic<size_t> packed[UP_SLOTS];
    for (auto &p : packed) p = 0;
    std::atomic<bool> stop{false};
    auto worker = [&] {
        for (;;) {
            const size_t job = next.fetch_add(1), k = job % UP_SLOTS;
            if (job >= up.jobs) return;
            while (open.load(std::memory_order_acquire) <= job) {
                if (stop) return;
                std::this_thread::yield();
            }
            up.pack(job, lo + k * UP_LO, hi + k * UP_HI);
            packed[k].fetch_add(1, std::memory_order_release);
        }
    };
    auto is_packed = [&](size_t job) { return packed[job % UP_SLOTS].load(std::memory_order_acquire) > job / UP_SLOTS; };
    std::thread t[UP_THREADS];
    int started = 0;
    try {
        for (; !failed && started < threads; started++) t[started] = std::thread(worker);
    } catch (...) {   // fewer threads then
    }
    for (size_t job = 0; job < up.jobs && !failed;) {
        // at most half of the ring is under way: the slots of the jobs up to half a ring ahead are free or soon will be
        const size_t upto = std::min(up.jobs, std::max(UP_SLOTS, job + UP_SLOTS / 2));
        for (size_t o = open.load(); o < upto && !failed; o++) {
            failed = !sg.wait(o % UP_SLOTS);
            open.store(o + 1, std::memory_order_release);
        }
        if (failed) break;
        const size_t k = job % UP_SLOTS;
        // one kind of job per copy, and no copy round the end of the ring
        const size_t most = std::min({up.jobs - job, job < up.off_jobs ? up.off_jobs - job : up.jobs, UP_SLOTS - k, UP_RUN_MOST});
        size_t n = 0;
        if (started == 0) {
            up.pack(job, lo + k * UP_LO, hi + k * UP_HI);
            n = 1;
        } else {
            while (n < std::min(most, UP_RUN)) {
                if (is_packed(job + n)) n++;
                else std::this_thread::yield();
            }
            while (n < most && is_packed(job + n)) n++;
        }
        if (up.copy(job, n, lo + k * UP_LO, hi + k * UP_HI, d_lo, d_hi, d_off, st) != hipSuccess ||
            hipEventRecord(sg.ev[k + n - 1], st) != hipSuccess)
            failed = true;
        for (size_t i = 0; i < n && !failed; i++) sg.copy_of[k + i] = (int)(k + n - 1);
        job += n;
    }
    stop = true;
    for (int w = 0; w < started; w++) t[w].join();
    if (failed) {
        (void)hipGetLastError();
        return PPV_EDEVICE;
    }
    if (up.invalid || up.longest > 0x7FFFFFFF) return PPV_EINVAL;
    *l_max = (int32_t)up.longest.load();
    return PPV_OK;
}
