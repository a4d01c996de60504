// Device memory of resident indexes (see devmem.h).
#include "devmem.h"

#include <unistd.h>

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <exception>
#include <mutex>
#include <new>
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
    enum State {
        idle,     // may be handed out again
        leaving,  // its caller waits for the kernels that may use it
        refused,  // not known to be idle
    } state;
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
    size_t unasked = 0;                      // bytes kept since the device was last asked what is free
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
            if (kept[i].state == Block::leaving || !which(kept[i])) {
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
            cv.wait_for(lk, std::chrono::milliseconds(250));
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

// Bytes that may stay kept on the current device, of which `more` are new.
size_t keep_limit(Keeper &k, size_t more) {
    k.unasked += more;
    if (k.unasked <= kKeepFreely) return kKeepBytes;
    k.unasked = 0;
    size_t free_bytes = 0, total = 0;
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess) return 0;
    return std::min(kKeepBytes, free_bytes / 4);
}

}  // namespace

hipError_t dev_malloc(void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    int device = 0;
    if (e != hipErrorOutOfMemory || hipGetDevice(&device) != hipSuccess) return e;
    (void)hipGetLastError();
    (void)dev_trim(device);  // (and waits for what its thread is just giving back)
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
            if (b.device == device && b.state == Block::idle && b.bytes >= bytes && b.bytes - bytes <= bytes / 8 &&
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
        k.used.emplace(*p, Block{*p, bytes, device, Clock::time_point(), Block::idle});
        ++k.blocks;
    } catch (const std::bad_alloc &) {
        (void)hipFree(*p);
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipSuccess;
}

void dev_free(std::initializer_list<void *> ps) {
    Keeper &k = keeper();
    int device = -1;
    {
        std::lock_guard<std::mutex> lk(k.mu);
        for (void *p : ps) {
            auto it = k.used.find(p);
            if (it == k.used.end()) continue;
            Block b = it->second;
            k.used.erase(it);
            b.state = Block::leaving;
            k.kept.push_back(b);
            device = b.device;
        }
    }
    if (device < 0) return;
    Current c(device);
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    std::lock_guard<std::mutex> lk(k.mu);
    size_t bytes = 0;
    for (Block &b : k.kept)
        if (std::find(ps.begin(), ps.end(), b.p) != ps.end()) {
            b.state = idle ? Block::idle : Block::refused;
            b.since = Clock::now();
            bytes += b.bytes;
        }
    const size_t limit = k.closing || !idle ? 0 : keep_limit(k, bytes);
    // those that have no room by themselves go, then the oldest until the rest have
    // (refused, they stay and are tried again)
    k.release([&](const Block &b) { return b.bytes > limit && std::find(ps.begin(), ps.end(), b.p) != ps.end(); });
    if (limit) {
        size_t over = k.held(device);
        over = over > limit ? over - limit : 0;
        k.release([&](const Block &b) {
            if (b.device != device || over == 0) return false;
            over -= std::min(over, b.bytes);
            return true;
        });
    }
    if (k.watching || k.closing || k.kept.empty()) return;
    if (k.watch.joinable()) k.watch.join();  // it has ended, or ends without the lock
    try {
        k.watch = std::thread([&k] { k.run(); });
        k.watching = true;
    } catch (const std::exception &) {
        k.release([&](const Block &b) { return b.device == device; });  // nobody would give them back
    }
}

size_t dev_kept(int device) {
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lk(k.mu);
    return k.held(device);
}

size_t dev_trim(int device) {
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lk(k.mu);
    const size_t before = k.held(device);
    k.release([&](const Block &b) { return b.device == device; });
    return before - k.held(device);
}

}  // namespace samatch
