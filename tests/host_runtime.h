// A stand-in for the HIP runtime on the CPU: the functions that libhisq.so
// imports, defined in the test program, take the place of the runtime's.
// Device memory is host memory, copies happen at once, a kernel launch only
// leaves work pending on the current device.  What the library's host code asks
// of the runtime, in which order and on which device, can be checked that way,
// error paths and a second device among it.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <sys/syscall.h>
#include <time.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>

namespace fake {

struct Block {
    size_t bytes;
    int device;
    long serial;
};

inline std::map<void *, Block> blocks;
inline long mallocs = 0, frees = 0, refused = 0, serial = 0;
inline size_t total = 0, max_block = ~(size_t)0, budget = ~(size_t)0;
inline bool free_fails = false, sync_fails = false;
inline long pending[2] = {0, 0};  // launches that nothing has waited for, per device
inline double clock_shift = 0.0;  // seconds added to the monotonic clock
inline dim3 last_grid, last_block;
inline float (*launch_ms)(dim3 grid, dim3 block) = nullptr;  // "time" of a launch, for events

inline thread_local int device = 0;
inline thread_local hipError_t last = hipSuccess;  // kept until hipGetLastError, as of ROCm 7
inline thread_local dim3 cfg_grid, cfg_block;
inline thread_local size_t cfg_shared;
inline thread_local hipStream_t cfg_stream;

inline hipError_t fail(hipError_t e) { return last = e; }

inline void *take(size_t n) {  // large blocks are address space only
    if (n < ((size_t)1 << 28)) return std::calloc(1, n + 256);
    void *p = mmap(nullptr, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p == MAP_FAILED ? nullptr : p;
}

// A small block is not given back, so that no two blocks ever have one address.
inline void give(void *p, size_t n) {
    if (n >= ((size_t)1 << 28)) munmap(p, n);
}

}  // namespace fake

extern "C" {

hipError_t hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (n > fake::max_block || fake::total + n > fake::budget) {
        ++fake::refused;
        return fake::fail(hipErrorOutOfMemory);
    }
    *p = fake::take(n);
    if (!*p) return fake::fail(hipErrorOutOfMemory);
    fake::blocks[*p] = {n, fake::device, fake::serial++};
    fake::total += n;
    ++fake::mallocs;
    return hipSuccess;
}

hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    if (fake::free_fails) return fake::fail(hipErrorStreamCaptureUnsupported);
    auto it = fake::blocks.find(p);
    if (it == fake::blocks.end()) {
        std::fprintf(stderr, "hipFree of %p, which is no block\n", p);
        std::exit(1);
    }
    fake::pending[it->second.device] = 0;  // waits for the block's device
    fake::total -= it->second.bytes;
    fake::give(p, it->second.bytes);
    fake::blocks.erase(it);
    ++fake::frees;
    return hipSuccess;
}

hipError_t hipGetDevice(int *d) { return *d = fake::device, hipSuccess; }
hipError_t hipSetDevice(int d) { return fake::device = d, hipSuccess; }
hipError_t hipDeviceSynchronize() {
    if (fake::sync_fails) return fake::fail(hipErrorStreamCaptureUnsupported);
    return fake::pending[fake::device] = 0, hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = fake::last;
    fake::last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
    fake::cfg_grid = grid;
    fake::cfg_block = block;
    fake::cfg_shared = shared;
    fake::cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
    *grid = fake::cfg_grid;
    *block = fake::cfg_block;
    *shared = fake::cfg_shared;
    *s = fake::cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t, hipStream_t) {
    ++fake::pending[fake::device];
    fake::last_grid = grid;
    fake::last_block = block;
    return hipSuccess;
}

hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    return std::memmove(d, s, n), hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)std::malloc(8), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return fake::pending[fake::device] = 0, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)std::malloc(8), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = fake::launch_ms ? fake::launch_ms(fake::last_grid, fake::last_block) : 1.f;
    return hipSuccess;
}

int clock_gettime(clockid_t id, struct timespec *t) {
    const long rc = syscall(SYS_clock_gettime, id, t);
    if (id == CLOCK_MONOTONIC) t->tv_sec += (time_t)fake::clock_shift;
    return (int)rc;
}

}  // extern "C"
