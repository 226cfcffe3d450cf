"""The memory that is kept between index builds, and the upload of a set (csrc/ppv_pool.hip): host code, built here with the
system's C++ compiler against a handful of HIP calls that work on host memory, with blocks kept for 200 ms.  Every case is a run
of its own, so that each also sees the process end with whatever it left."""
import os
import shutil
import subprocess

import pytest

from paper_2504_09135_amd import build as B

DRIVER = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <sys/wait.h>
#include <thread>
#include <unistd.h>
#include <vector>

#include "ppv_internal.h"

namespace {
std::mutex mu;
std::set<void *> live, pinned;
std::atomic<int> mallocs{0}, frees{0}, refuse_free{0}, refuse_pinned{0}, out_of_memory{0}, bad_mode{0};
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t) {
    std::lock_guard<std::mutex> l(mu);
    if (out_of_memory && !live.empty()) return hipErrorOutOfMemory;   // as long as anything is allocated
    *p = malloc(64);
    live.insert(*p);
    mallocs++;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> l(mu);
    if (mode != hipStreamCaptureModeRelaxed) bad_mode++;
    if (refuse_free) return hipErrorUnknown;
    if (!live.erase(p)) abort();
    free(p);
    frees++;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    std::lock_guard<std::mutex> l(mu);
    if (refuse_pinned && n > 1000000) return hipErrorOutOfMemory;
    *p = malloc(n);
    pinned.insert(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> l(mu);
    if (!pinned.erase(p)) abort();
    free(p);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, mode); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
}

#define CHECK(x) do { if (!(x)) { printf("%s:%d: %s\n", __FILE__, __LINE__, #x); fflush(stdout); _exit(1); } } while (0)
void sleep_ms(int ms) { std::this_thread::sleep_for(std::chrono::milliseconds(ms)); }
// waits for what a thread does in its own time, on a machine that may be busy
template <typename F> bool comes(F f) {
    for (int i = 0; i < 2000; i++) {
        if (f()) return true;
        sleep_ms(5);
    }
    return false;
}
size_t n_live() { std::lock_guard<std::mutex> l(mu); return live.size(); }
size_t n_pinned() { std::lock_guard<std::mutex> l(mu); return pinned.size(); }
constexpr size_t MB = 1 << 20;
void *take(size_t n) {
    void *p = nullptr;
    size_t got = 0;
    CHECK(ppv_pool_take(&p, n, &got) == PPV_OK && p && got >= n);
    return p;
}
void upload(unsigned seed, int64_t n, int32_t vocab, int times = 1) {
    std::vector<int64_t> off(n + 1);
    std::vector<int32_t> tok;
    for (int64_t i = 0; i < n; i++) {
        for (int k = (int)(seed + i) % 7 + 1; k > 0; k--) tok.push_back((int32_t)((tok.size() * 2654435761u + seed) % vocab));
        off[i + 1] = (int64_t)tok.size();
    }
    while (times-- > 0) {
        std::vector<uint16_t> lo(tok.size());
        std::vector<uint8_t> hi(vocab > 65536 ? tok.size() : 0);
        std::vector<uint32_t> o(n + 1);
        int32_t l_max = 0;
        CHECK(ppv_upload_set(tok.data(), off.data(), n, vocab, lo.data(), hi.empty() ? nullptr : hi.data(), o.data(), nullptr, &l_max) == PPV_OK);
        CHECK(l_max == 7);
        for (int64_t i = 0; i <= n; i++) CHECK(o[i] == (uint32_t)off[i]);
        for (size_t i = 0; i < tok.size(); i++) CHECK((uint32_t)tok[i] == (lo[i] | (hi.empty() ? 0u : (uint32_t)hi[i] << 16)));
    }
}

int main(int argc, char **argv) {
    const std::string which = argv[1];
    if (which == "reused") {
        void *a = take(3 * MB), *b = take(MB);
        ppv_pool_give(a, true);
        ppv_pool_give(b, true);
        CHECK(take(MB) == b && take(3 * MB - 5) == a && mallocs == 2 && frees == 0);   // (well within the 200 ms)
        ppv_pool_give(a, true);
        CHECK(take(MB) != a);          // much too large
        ppv_pool_give(b, false);       // (its wait failed)
        CHECK(frees == 1);
    } else if (which == "given_back") {   // without another call
        for (int round = 0; round < 3; round++) {
            void *a = take(3 * MB), *b = take(MB);
            ppv_pool_give(a, true);
            ppv_pool_give(b, true);
            CHECK(comes([] { return n_live() == 0; }));
            if (round == 1) sleep_ms(300);
        }
        upload(1, 1000, 300);
        CHECK(n_pinned() == 1);
        CHECK(comes([] { return n_pinned() == 0; }));
        upload(2, 1000, 300);
        CHECK(n_pinned() == 1);
    } else if (which == "refused") {      // a block that cannot be freed is not lost
        void *a = take(MB);
        refuse_free = 1;
        ppv_pool_give(a, true);
        sleep_ms(300);
        ppv_pool_empty();
        CHECK(n_live() == 1 && take(MB) == a);
        ppv_pool_give(a, true);
        refuse_free = 0;
        CHECK(comes([] { return n_live() == 0; }));
    } else if (which == "bounded") {
        void *p[5];
        for (void *&q : p) q = take(300 * MB);
        for (void *q : p) ppv_pool_give(q, true);
        CHECK(n_live() == 3);             // 1 GB
        void *q = take(1100 * MB);
        ppv_pool_give(q, true);
        CHECK(n_live() == 3);
        out_of_memory = 1;
        q = take(500 * MB);               // what is kept goes first
        CHECK(n_live() == 1);
        void *r;
        CHECK(ppv_pool_take(&r, MB) == PPV_ENOMEM && !r);
        ppv_pool_give(q, true);
        ppv_pool_empty();
        CHECK(n_live() == 0);
    } else if (which == "no_pinned") {
        refuse_pinned = 1;
        upload(1, 300000, 300);
        upload(2, 300000, 70000);
        sleep_ms(500);
        refuse_pinned = 0;
        upload(3, 300000, 70000);
        CHECK(n_pinned() == 1);
    } else if (which == "words") {        // the 65th waits
        std::vector<void *> w;
        for (int i = 0; i < 64; i++) w.push_back(ppv_host_words_take());
        CHECK(std::set<void *>(w.begin(), w.end()).size() == 64);
        std::atomic<void *> got{nullptr};
        std::thread t([&] { got = ppv_host_words_take(); });
        sleep_ms(50);
        CHECK(!got);
        ppv_host_words_give(w[37]);
        t.join();
        CHECK(got == w[37]);
    } else if (which == "threads") {
        std::vector<std::thread> t;
        for (int i = 0; i < 6; i++)
            t.emplace_back([i] {
                for (int k = 0; k < 30; k++) {
                    void *a = take((i + 1) * MB), *b = take(2 * MB), *w = ppv_host_words_take();
                    upload(i * 100 + k, 200000 + 10000 * i, i % 2 ? 300 : 70000);
                    if (k % 10 == 9) sleep_ms(90 * (i + 1));
                    ppv_host_words_give(w);
                    ppv_pool_give(a, true);
                    ppv_pool_give(b, true);
                }
            });
        for (auto &x : t) x.join();
        CHECK(comes([] { return n_live() == 0 && n_pinned() == 1; }));   // (the words)
    } else if (which == "child") {        // a forked child has neither the thread nor its wait at the end
        ppv_pool_give(take(MB), true);
        sleep_ms(20);
        const pid_t c = fork();
        if (c == 0) exit(7);
        int st = 0;
        CHECK(waitpid(c, &st, 0) == c && WIFEXITED(st) && WEXITSTATUS(st) == 7);
    } else {
        return 2;
    }
    CHECK(bad_mode == 0 && mode == hipStreamCaptureModeGlobal);
    printf("ok\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if not cxx:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("pool")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__=1", "-DPPV_POOL_AGE_MS=200",
                    "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-I", os.path.join(B.ROOT, "include"),
                    "-I", B.CSRC, "-x", "c++", os.path.join(B.CSRC, "ppv_pool.hip"), str(d / "driver.cpp"),
                    "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("case", ["reused", "given_back", "refused", "bounded", "no_pinned", "words", "threads", "child"])
def test_kept_memory(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.returncode, r.stdout, r.stderr)
