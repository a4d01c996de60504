// CPU check of what a device index build needs of device memory: the HIP
// functions that it calls are stood in for here, by a device of a given
// size whose kernels do nothing (the text then has no byte that is not a
// base, and no two suffixes share their first bases).
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "samatch.h"

namespace {
size_t device_bytes = (size_t)1 << 40, in_use = 0, most = 0;
std::map<void *, size_t> blocks;
}  // namespace

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 160 * 1024; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
    *free_bytes = device_bytes - in_use;
    *total = device_bytes;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
    if (in_use + bytes > device_bytes) return hipErrorOutOfMemory;
    *p = std::calloc(1, bytes);
    blocks[*p] = bytes;
    in_use += bytes;
    if (in_use > most) most = in_use;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    in_use -= blocks.at(p);
    blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { *p = std::calloc(1, bytes); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(to, from, n);
    return hipSuccess;
}
}

int main() {
    int failures = 0, limited = 0;
    for (int64_t n : {5'000, 100'000, 1'000'000, 3'000'000}) {
        const std::string text((size_t)n, 'A');
        sa_dindex *d = nullptr;
        device_bytes = (size_t)1 << 40;
        if (sa_build_device(text.data(), n, 0, &d) != SA_OK) return std::printf("FAIL: %s\n", sa_last_error()), 1;
        int64_t part[5];
        sa_dindex_bytes(d, part);
        const int64_t full = part[3];
        const size_t index = in_use - (((size_t)full + 255) & ~(size_t)255);
        sa_dfree(d);
        sa_trim(0, nullptr);
        if (in_use) return std::printf("FAIL: %zu bytes left\n", in_use), 1;
        // what the suffix sort works in: 36 bytes a base, histograms of 256 words per 2048 and a few words per 4096
        const size_t sort = 36 * (size_t)n + 1024 * ((size_t)n / 2048 + 1) + 8 * ((size_t)n / 4096 + 1) + 16 * 256 + 1024;
        // with the index and the sort it is enough; the table then takes a quarter of what is free at most
        for (size_t more = 0; more < 8 * sort; more += sort / 16) {
            device_bytes = index + sort + more;
            most = 0;
            if (sa_build_device(text.data(), n, 0, &d) != SA_OK) {
                std::printf("FAIL: %lld bases, %zu bytes besides index and sort: %s\n", (long long)n, more, sa_last_error());
                failures++;
                continue;
            }
            sa_dindex_bytes(d, part);
            limited += part[3] < full;
            if (4 * (size_t)part[3] > device_bytes - index) {
                std::printf("FAIL: %lld bases: a table of %lld bytes\n", (long long)n, (long long)part[3]);
                failures++;
            }
            sa_dfree(d);
            sa_trim(0, nullptr);
        }
        // without room for the sort the build fails, and gives everything back
        device_bytes = index + sort / 2;
        if (sa_build_device(text.data(), n, 0, &d) != SA_EDEVICE || (sa_trim(0, nullptr), in_use)) {
            std::printf("FAIL: %lld bases in too little memory, %zu bytes left\n", (long long)n, in_use);
            failures++;
        }
    }
    if (!limited) std::printf("FAIL: no build was short of memory\n"), failures++;
    std::printf("%s\n", failures ? "FAIL" : "ok");
    std::fflush(stdout);
    std::_Exit(failures ? 1 : 0);  // (without the exit handlers of the HIP runtime, which has no device here)
}
