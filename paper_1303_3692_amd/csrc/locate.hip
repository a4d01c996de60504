// Locate: the text positions of each read's occurrences, i.e. the suffix
// array entries of its row interval (Section IV lists the occurrences of a
// read this way, in suffix-array order), as a CSR list.
//
//   count    each read emits the first rows of [lo, hi) (at most cap), 0 for
//            reads not selected; bad intervals raise a flag instead of being
//            read.  Per-tile sums
//   emit     each workgroup adds up the tiles before its own (a scan kernel
//            does it for all when there are thousands) and all of them; then
//            the int64 offsets by a scan of the tile's reads and, when the
//            whole list fits the caller's buffer, SA[lo .. lo + count) of each
//            read, one thread per position
//   done     the total to the host, when the lists are written
//
// The host waits for the total in memory that the device writes over the bus.
// Bound by launches and that wait for batches of up to about a million
// reads: with a scratch of its own for each call and five device
// operations it took 98 us for 1,000,000 reads of 16 Mbp, now 30 (24 with the
// total handed over by the emit kernel, before the lists are whole).
#include <hip/hip_runtime.h>

#include <chrono>
#include <thread>

#include "device_state.h"
#include "devmem.h"

namespace samatch {

// Device words after the tile sums: the total, and the number of the last call with a bad interval.
constexpr int kLocTail = 2;
// Tiles up to which each workgroup adds up the sums by itself.
constexpr int kLocOwnSums = 2048;

LocateScratch::~LocateScratch() {
    if (dev) (void)hipFree(dev);
    if (host) (void)hipHostFree(host);
}

int LocateScratch::reserve(int64_t ntiles) {
    hipError_t e = hipSuccess;
    if (!host) {
        if ((e = hipHostMalloc((void **)&host, sizeof(LocateTotal), hipHostMallocMapped | hipHostMallocCoherent)) !=
                hipSuccess ||
            (e = hipHostGetDevicePointer((void **)&host_dev, host, 0)) != hipSuccess)
            return hip_fail(e, "locate scratch");
        host->call = 0;
    }
    if (ntiles > cap) {
        if (dev) (void)hipFree(dev);
        dev = nullptr;
        cap = 0;
        const int64_t c = std::max<int64_t>(ntiles, 256), zero[kLocTail] = {};
        if ((e = dev_malloc((void **)&dev, sizeof(int64_t) * (size_t)(c + kLocTail))) != hipSuccess ||
            (e = hipMemcpy(dev + c, zero, sizeof zero, hipMemcpyHostToDevice)) != hipSuccess)
            return hip_fail(e, "locate scratch");
        cap = c;
    }
    return SA_OK;
}

namespace {

constexpr int kLocBlock = 256;
// Rounds of kLocBlock reads per tile: few, so that a batch has workgroups for
// every compute unit (a tile's rounds follow each other: 1,000,000 reads took
// 30 us to emit in 245 tiles of 16 rounds, 12 in 977 of 4), and more once
// there are thousands of tiles, whose sums one workgroup adds up.
inline int loc_rounds(int64_t nreads) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(16, nreads / ((int64_t)kLocBlock * 1024)));
}

__device__ __forceinline__ int64_t read_count(const int4 h, int n, int cap, int min_len, bool &bad) {
    const bool sel = min_len > 0 ? (h.z >= min_len) : ((h.w & (int)SA_HIT_EXACT) != 0);
    if (!sel) return 0;
    if (h.x < 0 || h.y > n || h.x > h.y) {
        bad = true;
        return 0;
    }
    const int c = h.y - h.x;
    return c < cap ? c : cap;
}

// Block-wide inclusive sum of one int64 per thread; returns the total.
__device__ __forceinline__ int64_t block_incl_sum(int64_t v, int64_t &incl, int64_t *lds /* >= blockDim/64 */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    int64_t before = 0, total = 0;
    for (int w = 0; w < nw; ++w) {
        const int64_t s = lds[w];
        if (w < wave) before += s;
        total += s;
    }
    incl = before + x;
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(kLocBlock) void locate_count_kernel(const int4 *__restrict__ hits, int64_t nreads, int n,
                                                                 int cap, int min_len, int64_t *__restrict__ tile_sum,
                                                                 int64_t *__restrict__ tail, int64_t call, int rounds) {
    __shared__ int64_t lds[kLocBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kLocBlock * rounds;
    int64_t s = 0;
    bool bad = false;
#pragma unroll 4
    for (int r = 0; r < rounds; ++r) {
        const int64_t i = base + r * kLocBlock + threadIdx.x;
        if (i < nreads) s += read_count(hits[i], n, cap, min_len, bad);
    }
    if (bad) tail[1] = call;
    int64_t incl;
    const int64_t total = block_incl_sum(s, incl, lds);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// One workgroup: tile sums become the sum of the tiles before; tail[0] the total.
__global__ __launch_bounds__(1024) void locate_scan_tiles_kernel(int64_t *tile_sum, int ntiles, int64_t *tail) {
    __shared__ int64_t lds[1024 / 64];
    int64_t carry = 0;
    for (int b0 = 0; b0 < ntiles; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int64_t v = b < ntiles ? tile_sum[b] : 0;
        int64_t incl;
        const int64_t t = block_incl_sum(v, incl, lds);
        if (b < ntiles) tile_sum[b] = carry + incl - v;
        carry += t;
    }
    if (threadIdx.x == 0) tail[0] = carry;
}

// Offsets of the tile's reads, and their positions when the list fits: the
// 256 reads of a round own a run of the list, and each thread finds the read
// of its positions there by a binary search in LDS, so that neighbouring
// threads write neighbouring positions whatever the reads' counts.
__global__ __launch_bounds__(kLocBlock) void locate_emit_kernel(const int4 *__restrict__ hits, int64_t nreads, int n,
                                                                int cap, int min_len,
                                                                const int64_t *__restrict__ tile_sum,
                                                                int64_t *tail, bool scanned, int64_t call,
                                                                int64_t capacity,
                                                                const int32_t *__restrict__ sa,
                                                                int64_t *__restrict__ offs, int32_t *__restrict__ pos,
                                                                int rounds) {
    __shared__ int64_t lds[kLocBlock / 64];
    __shared__ int64_t start[kLocBlock];
    __shared__ int lo[kLocBlock];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kLocBlock * rounds;
    const int4 none = make_int4(0, 0, -1, 0);
    int4 next = base + t < nreads ? hits[base + t] : none;
    int64_t carry = 0, total = 0;
    if (scanned) {
        carry = tile_sum[blockIdx.x];
        total = tail[0];
    } else {
        int64_t before = 0, all = 0, incl;
        for (int b = t; b < (int)gridDim.x; b += kLocBlock) {
            const int64_t v = tile_sum[b];
            all += v;
            if (b < (int)blockIdx.x) before += v;
        }
        carry = block_incl_sum(before, incl, lds);
        total = block_incl_sum(all, incl, lds);
    }
    const bool bad = tail[1] == call;
    if (!scanned && blockIdx.x == 0 && t == 0) tail[0] = total;
    const bool fits = !bad && total <= capacity;
    for (int r = 0; r < rounds && base + r * kLocBlock < nreads; ++r) {
        const int64_t i = base + r * kLocBlock + t;
        const int4 h = next;
        next = r + 1 < rounds && i + kLocBlock < nreads ? hits[i + kLocBlock] : none;
        bool unused = false;
        const int64_t c = i < nreads ? read_count(h, n, cap, min_len, unused) : 0;
        int64_t incl;
        const int64_t count = block_incl_sum(c, incl, lds);
        if (i < nreads) offs[i] = carry + incl - c;
        if (fits && count > 0) {
            start[t] = incl - c;
            lo[t] = h.x;
            __syncthreads();
            for (int64_t j = t; j < count; j += kLocBlock) {
                int at = 0;  // the last read that starts at or before j (it has positions: later ones start after j)
#pragma unroll
                for (int step = kLocBlock / 2; step > 0; step >>= 1)
                    if (start[at + step] <= j) at += step;
                pos[carry + j] = sa[lo[at] + (int)(j - start[at])];
            }
            __syncthreads();
        }
        carry += count;
    }
    if (blockIdx.x == gridDim.x - 1 && t == 0) offs[nreads] = carry;
}

// Tells the waiting host that the call's lists are written.  A launch of its
// own: whoever reads the offsets after the call returned, on whatever stream,
// finds them whole, and a caller that was refused may release its buffers.
__global__ void locate_done_kernel(const int64_t *__restrict__ tail, int64_t call, LocateTotal *host) {
    host->total = tail[0];
    host->bad = tail[1] == call;
    __threadfence_system();
    __hip_atomic_store(&host->call, (uint64_t)call, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Waits until the device has written this call's total, or the
// stream has stopped without it.
int wait_total(LocateScratch &sc, uint64_t call, hipStream_t s) {
    for (int64_t spin = 0;; ++spin) {
        if (__atomic_load_n(&sc.host->call, __ATOMIC_ACQUIRE) == call) return SA_OK;
        if ((spin & 1023) != 1023) continue;
        const hipError_t e = hipStreamQuery(s);
        if (e == hipErrorNotReady) {
            (void)hipGetLastError();
            if (spin > 100000) std::this_thread::sleep_for(std::chrono::microseconds(20));
            continue;
        }
        if (e != hipSuccess) return hip_fail(e, "locate counts");
        if (__atomic_load_n(&sc.host->call, __ATOMIC_ACQUIRE) == call) return SA_OK;
        return fail(SA_EDEVICE, "locate: no total from the device");
    }
}

}  // namespace

// sa_locate_dev on the given scratch, whose mutex is held.
int locate_on(const sa_dindex *d, LocateScratch &sc, const sa_hit *d_hits, int64_t nreads, int32_t cap,
              int32_t min_len, int64_t *d_offs, int32_t *d_pos, int64_t pos_capacity, hipStream_t s, int64_t *total) {
    const int rounds = loc_rounds(nreads);
    const int64_t tile = (int64_t)kLocBlock * rounds;
    const int64_t ntiles = nreads > 0 ? (nreads + tile - 1) / tile : 1;
    if (ntiles > INT32_MAX) return fail(SA_EINVAL, "too many reads");
    if (int rc = sc.reserve(ntiles)) return rc;
    const int4 *hits = reinterpret_cast<const int4 *>(d_hits);
    const int n = (int)d->n;
    int64_t *tail = sc.dev + sc.cap;
    const int64_t call = (int64_t)++sc.calls;
    const bool scan = ntiles > kLocOwnSums;
    hipLaunchKernelGGL(locate_count_kernel, dim3((unsigned)ntiles), dim3(kLocBlock), 0, s, hits, nreads, n, cap,
                       min_len, sc.dev, tail, call, rounds);
    if (scan)
        hipLaunchKernelGGL(locate_scan_tiles_kernel, dim3(1), dim3(1024), 0, s, sc.dev, (int)ntiles, tail);
    hipLaunchKernelGGL(locate_emit_kernel, dim3((unsigned)ntiles), dim3(kLocBlock), 0, s, hits, nreads, n, cap,
                       min_len, sc.dev, tail, scan, call, pos_capacity, d->d_sa, d_offs, d_pos, rounds);
    hipLaunchKernelGGL(locate_done_kernel, dim3(1), dim3(1), 0, s, tail, call, sc.host_dev);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "locate launch");
    if (int rc = wait_total(sc, (uint64_t)call, s)) return rc;
    *total = sc.host->total;
    if (sc.host->bad) return fail(SA_EINVAL, "a selected hit has an interval outside [0, n]");
    if (*total > pos_capacity) return fail(SA_ENOSPC, "positions buffer too small (see *total)");
    return SA_OK;
}

}  // namespace samatch

using namespace samatch;

extern "C" int sa_locate_dev(const sa_dindex *d, const sa_hit *d_hits, int64_t nreads, int32_t cap, int32_t min_len,
                             int64_t *d_offs, int32_t *d_pos, int64_t pos_capacity, void *hip_stream,
                             int64_t *total) {
    clear_error();
    if (!d || !d_offs || !total || (nreads > 0 && !d_hits)) return fail(SA_EINVAL, "NULL argument");
    if (nreads < 0 || cap < 0 || min_len < 0 || pos_capacity < 0) return fail(SA_EINVAL, "negative size");
    if (pos_capacity > 0 && !d_pos) return fail(SA_EINVAL, "NULL positions buffer");
    DeviceGuard g(d->device);
    if (!g.ok) return fail(SA_EDEVICE, "hipSetDevice failed");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    LocateScratch &sc = workspace_for(const_cast<sa_dindex *>(d), s)->locate;
    std::lock_guard<std::mutex> lk(sc.mu);
    return locate_on(d, sc, d_hits, nreads, cap, min_len, d_offs, d_pos, pos_capacity, s, total);
}

extern "C" int sa_locate(const sa_dindex *d, const sa_hit *hits, int64_t nreads, int32_t cap, int32_t min_len,
                         int64_t *offs, int32_t *pos, int64_t pos_capacity, int64_t *total) {
    clear_error();
    if (!d || !offs || !total || (nreads > 0 && !hits)) return fail(SA_EINVAL, "NULL argument");
    if (nreads < 0 || cap < 0 || min_len < 0 || pos_capacity < 0) return fail(SA_EINVAL, "negative size");
    if (pos_capacity > 0 && !pos) return fail(SA_EINVAL, "NULL positions buffer");
    DeviceGuard g(d->device);
    if (!g.ok) return fail(SA_EDEVICE, "hipSetDevice failed");
    // the index's scratch, or one of its own while another thread's call has that
    // (MI355X, one read, a call for the total and one for the list: 122 us, and
    // 156 with a scratch per call, whose pinned memory has to be allocated)
    LocateScratch own, &kept = const_cast<sa_dindex *>(d)->locate;
    std::unique_lock<std::mutex> lk(kept.mu, std::try_to_lock);
    LocateScratch &scratch = lk.owns_lock() ? kept : own;
    struct Buffers {  // (released, and the stream waited for, before the scratch is)
        sa_hit *hits = nullptr;
        int64_t *offs = nullptr;
        int32_t *pos = nullptr;
        hipStream_t s = nullptr;
        ~Buffers() {
            if (s) (void)hipStreamSynchronize(s);
            if (hits) (void)hipFree(hits);
            if (offs) (void)hipFree(offs);
            if (pos) (void)hipFree(pos);
            if (s) (void)hipStreamDestroy(s);
        }
    } b;
    hipError_t e;
    if ((e = hipStreamCreateWithFlags(&b.s, hipStreamNonBlocking)) != hipSuccess ||
        (e = dev_malloc((void **)&b.hits, sizeof(sa_hit) * (size_t)(nreads > 0 ? nreads : 1))) != hipSuccess ||
        (e = dev_malloc((void **)&b.offs, sizeof(int64_t) * (size_t)(nreads + 1))) != hipSuccess)
        return hip_fail(e, "locate buffers");
    if (nreads > 0 &&
        (e = hipMemcpyAsync(b.hits, hits, sizeof(sa_hit) * (size_t)nreads, hipMemcpyHostToDevice, b.s)) != hipSuccess)
        return hip_fail(e, "locate upload");
    // counts and offsets first; positions only when they fit
    int rc = locate_on(d, scratch, b.hits, nreads, cap, min_len, b.offs, nullptr, 0, b.s, total);
    if (rc != SA_OK && rc != SA_ENOSPC) return rc;
    if ((e = hipMemcpyAsync(offs, b.offs, sizeof(int64_t) * (size_t)(nreads + 1), hipMemcpyDeviceToHost, b.s)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(b.s)) != hipSuccess)
        return hip_fail(e, "locate download");
    if (*total == 0) return SA_OK;
    if (*total > pos_capacity) return fail(SA_ENOSPC, "positions buffer too small (see *total)");
    if ((e = dev_malloc((void **)&b.pos, sizeof(int32_t) * (size_t)*total)) != hipSuccess)
        return hip_fail(e, "locate buffers");
    rc = locate_on(d, scratch, b.hits, nreads, cap, min_len, b.offs, b.pos, *total, b.s, total);
    if (rc) return rc;
    if ((e = hipMemcpyAsync(pos, b.pos, sizeof(int32_t) * (size_t)*total, hipMemcpyDeviceToHost, b.s)) != hipSuccess ||
        (e = hipStreamSynchronize(b.s)) != hipSuccess)
        return hip_fail(e, "locate download");
    return SA_OK;
}
