// CPU check of the memory keeper (devmem.hip): the functions of the HIP
// runtime that it calls are stood in for here, by a device of a given size
// that counts its memory and can refuse.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

#include "devmem.h"

namespace {

std::mutex &mu = *new std::mutex;  // (used by threads that run while the process ends)
size_t device_bytes = (size_t)64 << 30, in_use = 0;
std::map<void *, size_t> &blocks = *new std::map<void *, size_t>;
int refuse_frees = 0;        // so many calls of hipFree fail
int frees = 0;
std::atomic<bool> slow_frees{false};     // hipFree takes a second before the memory is there
bool capturing = false;      // a stream is captured in global mode, by another thread
bool capture_valid = true;
thread_local hipStreamCaptureMode thread_mode = hipStreamCaptureModeGlobal;

// A call that a capture in global mode does not allow any thread.
bool refused_by_capture() {
    if (!capturing || thread_mode == hipStreamCaptureModeRelaxed) return false;
    capture_valid = false;
    return true;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() {
    std::lock_guard<std::mutex> lk(mu);
    return refused_by_capture() ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
    std::swap(*m, thread_mode);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
    std::lock_guard<std::mutex> lk(mu);
    *free_bytes = device_bytes - in_use;
    *total = device_bytes;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
    std::lock_guard<std::mutex> lk(mu);
    if (refused_by_capture()) return hipErrorStreamCaptureUnsupported;
    if (in_use + bytes > device_bytes) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    blocks[*p] = bytes;
    in_use += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (slow_frees) std::this_thread::sleep_for(std::chrono::seconds(1));
    std::lock_guard<std::mutex> lk(mu);
    ++frees;
    if (refused_by_capture()) return hipErrorStreamCaptureUnsupported;
    if (refuse_frees > 0) {
        --refuse_frees;
        return hipErrorUnknown;
    }
    in_use -= blocks.at(p);
    blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
}

using namespace samatch;

static int failures = 0;

static void expect(bool ok, const char *what) {
    if (!ok) {
        std::printf("FAIL: %s\n", what);
        failures++;
    }
}

static size_t used() {
    std::lock_guard<std::mutex> lk(mu);
    return in_use;
}

static void *block(size_t bytes) {
    void *p = nullptr;
    expect(dev_alloc(&p, bytes) == hipSuccess && p, "allocation");
    return p;
}

// Waits until nothing is in use, at most `seconds`.
static bool idle_within(double seconds) {
    for (int i = 0; i < seconds * 100; i++) {
        if (used() == 0) return true;
        std::this_thread::sleep_for(std::chrono::milliseconds(10));
    }
    return used() == 0;
}

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    const size_t GiB = (size_t)1 << 30;
    if (!std::strcmp(what, "kept")) {  // used again, then given back
        void *p = block(GiB);
        dev_free({p});
        expect(dev_kept(0) == GiB, "kept");
        expect(block(GiB) == p, "used again");
        dev_free({p});
        expect(idle_within(kKeepSeconds + 2.0) && dev_kept(0) == 0, "given back");
    } else if (!std::strcmp(what, "limit")) {  // no more than kKeepBytes are kept, the oldest go first
        void *p[4];
        for (void *&x : p) x = block(3 * GiB);
        for (void *x : p) dev_free({x});
        expect(dev_kept(0) == 6 * GiB && used() == 6 * GiB, "two of four blocks kept");
        expect(blocks.count(p[2]) && blocks.count(p[3]), "the last ones");
        dev_trim(0);
        expect(dev_kept(0) == 0 && used() == 0, "nothing after a trim");
    } else if (!std::strcmp(what, "refused")) {  // a block that hipFree refuses is not lost
        void *p = block(GiB);
        dev_free({p});
        {
            std::lock_guard<std::mutex> lk(mu);
            refuse_frees = 1;
        }
        std::this_thread::sleep_for(std::chrono::milliseconds(1000 * kKeepSeconds + 500));
        {
            std::lock_guard<std::mutex> lk(mu);
            expect(frees == 1, "tried once");
        }
        expect(dev_kept(0) == GiB, "still kept");
        expect(idle_within(kKeepSeconds + 2.0) && dev_kept(0) == 0, "given back when tried again");
        p = block(GiB);
        dev_free({p});
        {
            std::lock_guard<std::mutex> lk(mu);
            refuse_frees = 1;
        }
        dev_trim(0);
        expect(dev_kept(0) == GiB, "a refused trim keeps the block");
        dev_trim(0);
        expect(used() == 0, "the next one gives it back");
    } else if (!std::strcmp(what, "capture")) {  // a capture of another thread goes on while kept blocks are given back
        void *p = block(GiB);
        dev_free({p});
        {
            std::lock_guard<std::mutex> lk(mu);
            capturing = true;
        }
        expect(idle_within(kKeepSeconds + 2.0), "given back during the capture");
        std::lock_guard<std::mutex> lk(mu);
        expect(capture_valid, "the capture is still valid");
        capturing = false;
    } else if (!std::strcmp(what, "pressure")) {  // kept memory is there for every allocation of the library
        void *p = block(7 * GiB), *rest = nullptr, *q = nullptr;
        dev_free({p});
        expect(dev_malloc(&rest, 60 * GiB) == hipSuccess && dev_kept(0) == 0, "dev_malloc takes what is kept");
        expect(dev_malloc(&q, 5 * GiB) == hipErrorOutOfMemory, "and fails when there is no more");
        expect(hipFree(rest) == hipSuccess, "release");
        dev_free({block(3 * GiB)});
        p = block(62 * GiB);
        expect(dev_kept(0) == 0, "so does dev_alloc");
        dev_free({p});
        expect(used() == 0, "a block of more than kKeepBytes is not kept");
        // the keeper's thread is giving a block back while another is asked for
        dev_free({block(4 * GiB)});
        std::this_thread::sleep_for(std::chrono::milliseconds(1000 * kKeepSeconds - 100));
        slow_frees = true;
        std::this_thread::sleep_for(std::chrono::milliseconds(400));
        expect(dev_malloc(&q, 62 * GiB) == hipSuccess, "waits for what is being given back");
    } else if (!std::strcmp(what, "full")) {  // little of a nearly full device is kept
        void *rest = nullptr;
        expect(dev_malloc(&rest, 60 * GiB) == hipSuccess, "allocation");
        void *small = block(kKeepFreely / 2), *large = block(2 * GiB), *fits = block(GiB * 3 / 8);
        dev_free({small});
        expect(dev_kept(0) == kKeepFreely / 2, "a small block is kept");
        dev_free({large});
        expect(dev_kept(0) == kKeepFreely / 2, "one of more than a quarter of the free memory is not");
        dev_free({fits});
        expect(dev_kept(0) == kKeepFreely / 2 + GiB * 3 / 8, "one of less is");
        expect(dev_trim(0) == kKeepFreely / 2 + GiB * 3 / 8 && dev_kept(0) == 0, "a trim says what it gave back");
        small = block(kKeepFreely / 2), large = block(2 * GiB);
        dev_free({small, nullptr, large});
        expect(dev_kept(0) == kKeepFreely / 2, "of several blocks those that fit are kept");
    } else if (!std::strcmp(what, "exit")) {  // the process ends with blocks kept, while threads free more
        std::thread([] {
            for (;;) {
                void *p = nullptr;
                if (dev_alloc(&p, (size_t)1 << 20) == hipSuccess) dev_free({p});
            }
        }).detach();
        std::this_thread::sleep_for(std::chrono::milliseconds(100));
    } else {
        std::printf("no such check\n");
        return 1;
    }
    std::printf("%s\n", failures ? "FAIL" : "ok");
    std::fflush(stdout);
    return failures ? 1 : 0;
}
