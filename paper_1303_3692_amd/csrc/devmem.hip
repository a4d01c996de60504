// Device memory of resident indexes (see devmem.h).
#include "devmem.h"

#include <unistd.h>

#include <chrono>
#include <condition_variable>
#include <mutex>
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
    Clock::time_point since;  // when it was kept
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
    std::vector<Block> kept;
    std::thread watch;  // gives back what is not used again; ends when nothing is kept
    bool watching = false, closing = false;

    // The process ends, and its memory with it: nothing is kept any more.
    void close() {
        {
            std::lock_guard<std::mutex> lk(mu);
            closing = true;
        }
        cv.notify_all();
        if (watch.joinable()) watch.join();
    }

    static void release(const std::vector<Block> &blocks) {
        for (const Block &b : blocks) {
            Current c(b.device);
            (void)hipFree(b.p);
        }
    }

    std::vector<Block> take_kept(int device, Clock::time_point before) {
        std::vector<Block> out, stay;
        for (const Block &b : kept)
            ((device < 0 || b.device == device) && b.since <= before ? out : stay).push_back(b);
        kept.swap(stay);
        return out;
    }

    void run() {
        std::unique_lock<std::mutex> lk(mu);
        while (!closing && !kept.empty()) {
            Clock::time_point oldest = kept[0].since;
            for (const Block &b : kept) oldest = std::min(oldest, b.since);
            const Clock::time_point due = oldest + std::chrono::seconds(kKeepSeconds);
            if (Clock::now() < due) {
                cv.wait_until(lk, due);
                continue;
            }
            const std::vector<Block> old = take_kept(-1, Clock::now() - std::chrono::seconds(kKeepSeconds));
            lk.unlock();
            release(old);
            lk.lock();
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
            if (b.device == device && b.bytes >= bytes && b.bytes - bytes <= bytes / 8 &&
                (best == k.kept.size() || b.bytes < k.kept[best].bytes))
                best = i;
        }
        if (best < k.kept.size()) {
            const Block b = k.kept[best];
            k.kept.erase(k.kept.begin() + (long)best);
            k.used.emplace(b.p, b);
            *p = b.p;
            return hipSuccess;
        }
    }
    e = hipMalloc(p, bytes);
    if (e != hipSuccess && dev_kept(device) > 0) {
        (void)hipGetLastError();
        dev_trim(device);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(k.mu);
    k.used.emplace(*p, Block{*p, bytes, device, Clock::time_point()});
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
        k.used.erase(it);
    }
    Current c(b.device);
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    if (idle && !closing && b.bytes <= kKeepBytes) {
        std::vector<Block> out;  // the oldest ones, when there is no room for this one
        {
            std::lock_guard<std::mutex> lk(k.mu);
            size_t held = b.bytes;
            for (const Block &x : k.kept)
                if (x.device == b.device) held += x.bytes;
            for (size_t i = 0; i < k.kept.size() && held > kKeepBytes;) {
                if (k.kept[i].device != b.device) {
                    i++;
                    continue;
                }
                held -= k.kept[i].bytes;
                out.push_back(k.kept[i]);
                k.kept.erase(k.kept.begin() + (long)i);
            }
            b.since = Clock::now();
            k.kept.push_back(b);
            if (!k.watching) {
                if (k.watch.joinable()) k.watch.join();  // it has ended, or ends without the lock
                try {
                    k.watch = std::thread([&k] { k.run(); });
                    k.watching = true;
                } catch (const std::system_error &) {
                    out.push_back(k.kept.back());  // nobody would give it back
                    k.kept.pop_back();
                }
            }
        }
        Keeper::release(out);
        return;
    }
    (void)hipFree(b.p);
}

size_t dev_kept(int device) {
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lk(k.mu);
    size_t held = 0;
    for (const Block &b : k.kept)
        if (b.device == device) held += b.bytes;
    return held;
}

void dev_trim(int device) {
    Keeper &k = keeper();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> lk(k.mu);
        out = k.take_kept(device, Clock::time_point::max());
    }
    Keeper::release(out);
}

}  // namespace samatch
