// Device memory of resident indexes (see devmem.h).
#include "devmem.h"

#include <unistd.h>

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <unordered_map>
#include <vector>

namespace samatch {
namespace {

using Clock = std::chrono::steady_clock;

struct Block {
    void *p;
    size_t bytes;
    int device;
    Clock::time_point since;  // when it was kept, or last refused by hipFree
    bool idle;                // no kernel uses it: it may be handed out again
};

// Makes a device current for the scope.
struct Current {
    explicit Current(int device) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != device) (void)hipSetDevice(device);
    }
    ~Current() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
    int prev = -1;
};

struct Keeper {
    std::mutex mu;
    std::condition_variable cv;
    std::unordered_map<void *, Block> used;  // blocks handed out
    std::vector<Block> kept;                 // has room for every block there is, so that keeping one allocates nothing
    size_t blocks = 0;                       // there are: handed out, kept, or on their way
    std::thread watch;  // gives back what is not used again; ends when nothing is kept
    bool watching = false, closing = false;

    // The process ends, and its memory with it: nothing is kept any more.
    void close() {
        std::thread last;
        {
            std::lock_guard<std::mutex> lk(mu);
            closing = true;
            last.swap(watch);
        }
        cv.notify_all();
        if (last.joinable()) last.join();
    }

    // Gives those kept blocks back for which `which` holds (with the lock
    // held, so that whoever finds too little memory meanwhile waits for
    // this).  A block that hipFree refuses stays, and is tried again.
    template <class F>
    void release(F which) {
        for (size_t i = 0; i < kept.size();) {
            if (!which(kept[i])) {
                ++i;
                continue;
            }
            Current c(kept[i].device);
            if (hipFree(kept[i].p) == hipSuccess) {
                kept.erase(kept.begin() + (long)i);
                --blocks;
            } else {
                (void)hipGetLastError();
                kept[i].since = Clock::now();
                ++i;
            }
        }
    }

    size_t held(int device) const {
        size_t bytes = 0;
        for (const Block &b : kept)
            if (b.device == device) bytes += b.bytes;
        return bytes;
    }

    void run() {
        // another thread may be capturing a stream in global mode, which
        // forbids every thread a hipFree that has not asked for this mode
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        std::unique_lock<std::mutex> lk(mu);
        while (!closing && !kept.empty()) {
            Clock::time_point oldest = kept[0].since;
            for (const Block &b : kept) oldest = std::min(oldest, b.since);
            const Clock::time_point due = oldest + std::chrono::seconds(kKeepSeconds);
            if (Clock::now() < due) {
                cv.wait_until(lk, due);
                continue;
            }
            const Clock::time_point before = Clock::now() - std::chrono::seconds(kKeepSeconds);
            release([&](const Block &b) { return b.since <= before; });
        }
        watching = false;
    }
};

// Never destroyed, so that an index freed while the process ends finds it;
// its thread is ended before the HIP runtime is (which was loaded before).
// A forked child has no such thread to wait for.
Keeper &keeper() {
    static Keeper *k = new Keeper;
    static struct Closer {
        Keeper *k;
        pid_t owner;
        ~Closer() {
            if (getpid() == owner) k->close();
        }
    } closer{k, getpid()};
    return *k;
}

}  // namespace

hipError_t dev_malloc(void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    int device = 0;
    if (e != hipErrorOutOfMemory || hipGetDevice(&device) != hipSuccess) return e;
    (void)hipGetLastError();
    dev_trim(device);  // (and waits for what its thread is just giving back)
    return hipMalloc(p, bytes);
}

hipError_t dev_alloc(void **p, size_t bytes) {
    *p = nullptr;
    bytes = (bytes + 255) & ~(size_t)255;
    if (bytes == 0) bytes = 256;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    Keeper &k = keeper();
    {
        // the smallest kept block that holds it and wastes at most an eighth
        std::lock_guard<std::mutex> lk(k.mu);
        size_t best = k.kept.size();
        for (size_t i = 0; i < k.kept.size(); i++) {
            const Block &b = k.kept[i];
            if (b.device == device && b.idle && b.bytes >= bytes && b.bytes - bytes <= bytes / 8 &&
                (best == k.kept.size() || b.bytes < k.kept[best].bytes))
                best = i;
        }
        if (best < k.kept.size()) {
            const Block b = k.kept[best];
            try {
                k.used.emplace(b.p, b);
            } catch (const std::bad_alloc &) {
                return hipErrorOutOfMemory;
            }
            k.kept.erase(k.kept.begin() + (long)best);
            *p = b.p;
            return hipSuccess;
        }
    }
    if ((e = dev_malloc(p, bytes)) != hipSuccess) return e;
    try {
        std::lock_guard<std::mutex> lk(k.mu);
        k.kept.reserve(k.blocks + 1);
        k.used.emplace(*p, Block{*p, bytes, device, Clock::time_point(), true});
        ++k.blocks;
    } catch (const std::bad_alloc &) {
        (void)hipFree(*p);
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipSuccess;
}

void dev_free(void *p) {
    if (!p) return;
    Keeper &k = keeper();
    Block b;
    bool closing;
    {
        std::lock_guard<std::mutex> lk(k.mu);
        closing = k.closing;
        auto it = k.used.find(p);
        if (it == k.used.end()) return;
        b = it->second;
        k.used.erase(it);  // before hipFree, after which another thread may be given the same address
    }
    Current c(b.device);
    b.idle = hipDeviceSynchronize() == hipSuccess;
    if (!b.idle || closing || b.bytes > kKeepBytes) {
        if (hipFree(p) == hipSuccess) {
            std::lock_guard<std::mutex> lk(k.mu);
            --k.blocks;
            return;
        }
        (void)hipGetLastError();  // kept, and tried again
    }
    std::lock_guard<std::mutex> lk(k.mu);
    // the oldest ones go when there is no room for this one
    size_t held = k.held(b.device) + b.bytes;
    k.release([&](const Block &x) {
        if (x.device != b.device || held <= kKeepBytes) return false;
        held -= x.bytes;
        return true;
    });
    b.since = Clock::now();
    k.kept.push_back(b);
    if (k.watching || k.closing) return;
    if (k.watch.joinable()) k.watch.join();  // it has ended, or ends without the lock
    try {
        k.watch = std::thread([&k] { k.run(); });
        k.watching = true;
    } catch (const std::system_error &) {
        k.release([&](const Block &x) { return x.p == p; });  // nobody would give it back
    }
}

size_t dev_kept(int device) {
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lk(k.mu);
    return k.held(device);
}

void dev_trim(int device) {
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lk(k.mu);
    k.release([&](const Block &b) { return b.device == device; });
}

}  // namespace samatch
