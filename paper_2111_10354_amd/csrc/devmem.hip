// Device memory of the library's handles, workspaces and temporaries.
//
// Memory that hipMalloc hands out is cleared first, at 59 GB/s once the
// memory that the driver had cleared ahead is used up (after 288 GB in all).
// A program that makes and frees a handle or a workspace per gauge
// configuration comes to that point within a few hundred of them: a
// smearing of 48^3 x 12 with a fresh 1.1 GB workspace took 13 ms for 290
// calls, then 32 ms with some of 100 to 580 ms, and 12.7 ms every time with a
// kept one.  So blocks are kept for the next allocation of about their size:
//   * a block enters the list only through recycle(), which its owner calls
//     once all work on it has ended, so any stream and any thread may get it;
//     everywhere else (error paths among it) release() frees it;
//   * the list is bounded (kKeepBytes in all, kKeepBlocks), the oldest blocks
//     leaving first; a block over the bound is freed at once;
//   * a block that nobody wanted for kKeepSeconds is freed by the next call
//     that allocates or recycles, and all are freed when an allocation fails.

#include <chrono>
#include <list>

#include "solver_internal.h"

namespace hisq {

namespace {

typedef std::chrono::steady_clock Clock;

struct Block {
    void *p;
    size_t bytes;
    int device;
    Clock::time_point since;
};

constexpr size_t kKeepBytes = (size_t)16 << 30;  // 6 % of the device
constexpr size_t kKeepBlocks = 256;
constexpr double kKeepSeconds = 5.0;

struct Kept {
    std::mutex mu;
    std::list<Block> blocks;  // oldest first
    size_t total = 0;

    void drop(std::list<Block>::iterator it) {
        total -= it->bytes;
        (void)hipFree(it->p);
        blocks.erase(it);
    }
    void drop_old(Clock::time_point now) {
        while (!blocks.empty() && std::chrono::duration<double>(now - blocks.front().since).count() > kKeepSeconds)
            drop(blocks.begin());
    }
    // the smallest block of n to 9/8 n bytes (nullptr if none)
    void *take(size_t n, int device, size_t *bytes) {
        auto best = blocks.end();
        for (auto it = blocks.begin(); it != blocks.end(); ++it)
            if (it->device == device && it->bytes >= n && it->bytes - n <= n / 8 &&
                (best == blocks.end() || it->bytes < best->bytes))
                best = it;
        if (best == blocks.end()) return nullptr;
        void *p = best->p;
        *bytes = best->bytes;
        total -= best->bytes;
        blocks.erase(best);
        return p;
    }
};

// Never destroyed: the HIP runtime may be gone when static destructors run.
Kept &kept() {
    static Kept *k = new Kept();
    return *k;
}

}  // namespace

int DevBuf::alloc(size_t n) {
    if (p && bytes >= n) return HISQ_OK;
    release();
    if (n == 0) return HISQ_OK;
    int dev = -1;
    HISQ_HIP_CHECK(hipGetDevice(&dev));
    Kept &k = kept();
    {
        std::lock_guard<std::mutex> lk(k.mu);
        p = k.take(n, dev, &held);
        k.drop_old(Clock::now());
    }
    if (!p) {
        held = n;
        hipError_t e = hipMalloc(&p, n);
        if (e == hipErrorOutOfMemory) {
            std::lock_guard<std::mutex> lk(k.mu);
            if (!k.blocks.empty()) {
                while (!k.blocks.empty()) k.drop(k.blocks.begin());
                e = hipMalloc(&p, n);
            }
            // The runtime keeps a failed call's error until it is asked for it:
            // the check after the next launch must not find these.
            (void)hipGetLastError();
        }
        if (e != hipSuccess) {
            p = nullptr;
            set_error(std::string("hipMalloc(") + std::to_string(n) + "): " + hipGetErrorString(e));
            return e == hipErrorOutOfMemory ? HISQ_ERR_OOM : HISQ_ERR_HIP;
        }
    }
    bytes = n;
    device = dev;
    return HISQ_OK;
}

void DevBuf::release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = held = 0;
}

void DevBuf::recycle() {
    if (!p || held > kKeepBytes) return release();
    Kept &k = kept();
    const auto now = Clock::now();
    {
        std::lock_guard<std::mutex> lk(k.mu);
        while (!k.blocks.empty() && (k.total + held > kKeepBytes || k.blocks.size() >= kKeepBlocks))
            k.drop(k.blocks.begin());
        k.blocks.push_back({p, held, device, now});
        k.total += held;
        k.drop_old(now);
    }
    p = nullptr;
    bytes = held = 0;
}

}  // namespace hisq
