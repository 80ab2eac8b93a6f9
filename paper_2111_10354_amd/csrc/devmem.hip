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
//     that allocates or recycles, and all are freed when an allocation fails
//     or the program asks for it (release_kept);
//   * the list is a fixed array: giving a block back allocates nothing and
//     cannot fail.

#include <algorithm>
#include <chrono>
#include <new>

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
constexpr int kKeepBlocks = 256;
constexpr double kKeepSeconds = 5.0;

struct Kept {
    std::mutex mu;
    Block blocks[kKeepBlocks];  // the first n, oldest first
    int n = 0;
    size_t total = 0;

    void remove(int i) {
        total -= blocks[i].bytes;
        std::copy(blocks + i + 1, blocks + n, blocks + i);
        --n;
    }
    // false: the runtime refuses (while a thread captures a graph): the block stays
    bool drop(int i) {
        if (hipFree(blocks[i].p) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        remove(i);
        return true;
    }
    void drop_old(Clock::time_point now) {
        while (n > 0 && std::chrono::duration<double>(now - blocks[0].since).count() > kKeepSeconds && drop(0)) {
        }
    }
    bool drop_all() {
        while (n > 0 && drop(n - 1)) {
        }
        return n == 0;
    }
    // room for a block of b <= kKeepBytes bytes
    bool make_room(size_t b) {
        while (n > 0 && (total + b > kKeepBytes || n >= kKeepBlocks))
            if (!drop(0)) return false;
        return true;
    }
    // the smallest block of b to 9/8 b bytes (nullptr if none)
    void *take(size_t b, int device, size_t *bytes) {
        int best = -1;
        for (int i = 0; i < n; ++i)
            if (blocks[i].device == device && blocks[i].bytes >= b && blocks[i].bytes - b <= b / 8 &&
                (best < 0 || blocks[i].bytes < blocks[best].bytes))
                best = i;
        if (best < 0) return nullptr;
        void *p = blocks[best].p;
        *bytes = blocks[best].bytes;
        remove(best);
        return p;
    }
};

// Never destroyed: the HIP runtime may be gone when static destructors run.
Kept &kept() {
    alignas(Kept) static unsigned char mem[sizeof(Kept)];
    static Kept *k = new (mem) Kept();
    return *k;
}

}  // namespace

int release_kept(size_t *bytes) {
    Kept &k = kept();
    std::lock_guard<std::mutex> lk(k.mu);
    const size_t before = k.total;
    const bool all = k.drop_all();
    if (bytes) *bytes = before - k.total;
    if (all) return HISQ_OK;
    set_error("kept device memory could not be freed");
    return HISQ_ERR_HIP;
}

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
            if (k.n > 0) {
                (void)k.drop_all();
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
    if (p && hipFree(p) != hipSuccess) (void)hipGetLastError();
    p = nullptr;
    bytes = held = 0;
}

void DevBuf::recycle() {
    if (!p || held > kKeepBytes) return release();
    Kept &k = kept();
    const auto now = Clock::now();
    {
        std::lock_guard<std::mutex> lk(k.mu);
        if (!k.make_room(held)) return release();
        k.blocks[k.n++] = {p, held, device, now};
        k.total += held;
        k.drop_old(now);
    }
    p = nullptr;
    bytes = held = 0;
}

}  // namespace hisq
