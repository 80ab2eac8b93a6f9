// Host code of libhisq.so against the stand-in runtime of host_runtime.h (no
// GPU).  usage: host_runtime_check CASE; prints "ok", or what failed.
#include "host_runtime.h"

#include <array>
#include <new>
#include <string>
#include <vector>

#include "hisq.h"
#include "nn_internal.h"

using namespace hisq;

#define CHECK(cond)                                                       \
    do {                                                                  \
        if (!(cond)) {                                                    \
            std::printf("FAILED line %d: %s\n", __LINE__, #cond);         \
            std::exit(1);                                                 \
        }                                                                 \
    } while (0)

static hisq_gauge_t make_gauge(const int dims[4], unsigned precs) {
    static std::vector<double> links;  // zero: not compressible, small enough for FP16
    const size_t V = (size_t)dims[0] * dims[1] * dims[2] * dims[3];
    links.assign(V * 72, 0.0);
    hisq_gauge_t g = nullptr;
    CHECK(hisq_gauge_create(&g, dims, links.data(), links.data(), precs, nullptr) == HISQ_OK);
    return g;
}

// A handle of device 1 destroyed while device 0 is current: its blocks must not
// go to the next allocation there before device 1 has been waited for.
static void destroy_other_device() {
    const int dims[4] = {8, 8, 8, 8};
    hipSetDevice(1);
    hisq_gauge_t g = make_gauge(dims, HISQ_PREC_MASK(HISQ_PREC_FP32));
    std::vector<char> in(spinor_bytes(F32, 2048) + 16), out(in.size());
    auto align = [](std::vector<char> &v) { return (void *)(((uintptr_t)v.data() + 15) & ~(uintptr_t)15); };
    CHECK(hisq_dslash_eo(g, 0, HISQ_PREC_FP32, align(in), align(out), nullptr) == HISQ_OK);
    CHECK(fake::pending[1] > 0);
    hipSetDevice(0);
    CHECK(hisq_gauge_destroy(g) == HISQ_OK);
    int dev = -1;
    CHECK(hipGetDevice(&dev) == hipSuccess && dev == 0);
    CHECK(fake::pending[1] == 0);
}

// Training where memory for one sample's buffers is there and for a whole
// batch's is not: the batch trains, larger blocks are not asked for again and
// again, no failed allocation is left as the thread's last error, and the
// buffers that the network has are never given up for larger ones.
static void training_without_memory() {
    const int dims[4] = {8, 8, 8, 8}, ch[4] = {1, 8, 8, 1};
    hisq_gauge_t g = make_gauge(dims, HISQ_PREC_MASK(HISQ_PREC_FP32));
    std::vector<double> thin(4096 * 72, 0.0);
    CHECK(hisq_gauge_set_thin(g, thin.data(), nullptr) == HISQ_OK);
    hisq_nn_t net = nullptr;
    CHECK(hisq_nn_create(&net, g, 3, ch, nullptr, nullptr) == HISQ_OK);
    std::vector<float> v(8 * 6 * 2048 + 4, 0.f);
    double loss = -1.0;
    const size_t have = net->train.mem.bytes;
    CHECK(net->train.cap == 1 && have > 0);
    fake::max_block = have;
    for (int k = 0; k < 3; ++k) {
        CHECK(hisq_nn_loss_grad(net, 8, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
        CHECK(hisq_nn_train_step(net, 8, v.data(), v.data(), 1e-3, &loss, nullptr) == HISQ_OK);
        CHECK(net->train.mem.bytes >= have);
    }
    const long refused = fake::refused;
    CHECK(hisq_nn_loss_grad(net, 8, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
    CHECK(fake::refused == refused);
    fake::max_block = 6 * have;  // a smaller batch may ask again
    CHECK(hisq_nn_loss_grad(net, 3, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
    CHECK(net->train.cap >= 2);
    const size_t grown = net->train.mem.bytes;
    fake::max_block = 0;  // nothing: the buffers stay
    CHECK(hisq_nn_loss_grad(net, 8, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
    CHECK(net->train.mem.bytes == grown);
    fake::max_block = ~(size_t)0;
    CHECK(hisq_nn_destroy(net) == HISQ_OK && hisq_gauge_destroy(g) == HISQ_OK);
}

// Destroying while the runtime refuses to wait or to free (a thread captures a
// graph) leaves no error for the next launch check.
static void destroy_while_refused() {
    const int dims[4] = {8, 8, 8, 8}, ch[3] = {1, 8, 1};
    hisq_gauge_t g = make_gauge(dims, HISQ_PREC_MASK(HISQ_PREC_FP32));
    hisq_nn_t net = nullptr;
    CHECK(hisq_nn_create(&net, g, 2, ch, nullptr, nullptr) == HISQ_OK);
    fake::sync_fails = fake::free_fails = true;
    CHECK(hisq_nn_destroy(net) == HISQ_OK && hipGetLastError() == hipSuccess);
    CHECK(hisq_gauge_destroy(g) == HISQ_OK && hipGetLastError() == hipSuccess);
    fake::sync_fails = fake::free_fails = false;
    size_t freed = 1;
    CHECK(hisq_release_memory(&freed) == HISQ_OK && freed <= 8);  // nothing was kept of either
}

// A network's blocks go to the next one, once its device is idle.
static void network_blocks() {
    const int dims[4] = {8, 8, 8, 8}, ch[4] = {1, 8, 8, 1};
    hipSetDevice(1);
    hisq_gauge_t g = make_gauge(dims, HISQ_PREC_MASK(HISQ_PREC_FP32));
    std::vector<double> thin(4096 * 72, 0.0);
    CHECK(hisq_gauge_set_thin(g, thin.data(), nullptr) == HISQ_OK);
    void *in = (void *)((uintptr_t)1 << 40), *out = (void *)((uintptr_t)1 << 41);
    long mallocs = 0;
    for (int k = 0; k < 3; ++k) {
        hisq_nn_t net = nullptr;
        hipSetDevice(1);
        if (k == 1) mallocs = fake::mallocs;
        CHECK(hisq_nn_create(&net, g, 3, ch, nullptr, nullptr) == HISQ_OK);
        CHECK(hisq_precond_apply(g, net, in, out, nullptr) == HISQ_OK && fake::pending[1] > 0);
        hipSetDevice(0);
        CHECK(hisq_nn_destroy(net) == HISQ_OK);
        int dev = -1;
        CHECK(hipGetDevice(&dev) == hipSuccess && dev == 0 && fake::pending[1] == 0);
    }
    CHECK(fake::mallocs == mallocs);
    CHECK(hisq_gauge_destroy(g) == HISQ_OK);
}

// An allocation that fails, with or without kept blocks to give up, leaves no
// error behind: the next launch check is not the one to report it.
static void failed_allocation() {
    for (int kept = 0; kept < 2; ++kept) {
        if (kept) {
            DevBuf k;
            CHECK(k.alloc(1 << 20) == HISQ_OK);
            k.recycle();
        }
        fake::max_block = 1 << 21;
        DevBuf b;
        CHECK(b.alloc(1 << 22) == HISQ_ERR_OOM);
        CHECK(hipGetLastError() == hipSuccess);
        fake::max_block = ~(size_t)0;
        CHECK(b.alloc(1 << 22) == HISQ_OK);
    }
}

// The list of kept blocks: what it hands on, and when it frees.
static void kept_blocks() {
    const size_t M = 1 << 20;
    auto keep = [](size_t n) {
        DevBuf b;
        CHECK(b.alloc(n) == HISQ_OK);
        void *p = b.p;
        b.recycle();
        CHECK(!b.p && !b.bytes);
        return p;
    };
    // a block goes to an allocation of 8/9 of its size to its own, on its device
    void *p = keep(9 * M);
    const long mallocs = fake::mallocs;
    {
        DevBuf a, b, c;
        CHECK(a.alloc(8 * M - 1) == HISQ_OK && a.p != p);
        CHECK(b.alloc(9 * M + 1) == HISQ_OK && b.p != p);
        hipSetDevice(1);
        CHECK(c.alloc(9 * M) == HISQ_OK && c.p != p);
        hipSetDevice(0);
        CHECK(fake::mallocs == mallocs + 3);
        DevBuf d;
        CHECK(d.alloc(8 * M) == HISQ_OK && d.p == p && d.bytes == 8 * M && fake::mallocs == mallocs + 3);
        d.recycle();
        CHECK(d.alloc(9 * M) == HISQ_OK && d.p == p);  // still the whole block
    }
    // the smallest of several that fit
    {
        void *large = keep(10 * M);
        DevBuf s;
        CHECK(s.alloc(9 * M + M / 2) == HISQ_OK && s.p == large);
        DevBuf t;
        CHECK(t.alloc(9 * M + M / 4) == HISQ_OK);
        void *small = t.p;
        s.recycle();
        t.recycle();
        DevBuf u;
        CHECK(u.alloc(9 * M) == HISQ_OK && u.p == small);
    }
    size_t freed = 0;
    CHECK(hisq_release_memory(&freed) == HISQ_OK && freed == 10 * M);
    CHECK(hisq_release_memory(&freed) == HISQ_OK && freed == 0 && fake::blocks.empty());

    // at most 16 GiB and 256 blocks, the oldest leaving first; larger ones at once
    const size_t G = (size_t)1 << 30;
    keep(17 * G);
    CHECK(fake::total == 0);
    void *first = keep(3 * G);
    void *second = keep(6 * G);
    void *third = keep(9 * G);
    CHECK(!fake::blocks.count(first) && fake::blocks.count(second) && fake::blocks.count(third));
    CHECK(hisq_release_memory(nullptr) == HISQ_OK && fake::total == 0);
    {
        std::vector<DevBuf> many(257);
        for (auto &b : many) CHECK(b.alloc(4096) == HISQ_OK);
        first = many[0].p;
        second = many[1].p;
        for (auto &b : many) b.recycle();
    }
    CHECK(fake::blocks.size() == 256 && !fake::blocks.count(first) && fake::blocks.count(second));
    CHECK(hisq_release_memory(nullptr) == HISQ_OK && fake::total == 0);

    // after five seconds the next call that allocates or recycles frees it
    p = keep(M);
    fake::clock_shift += 4.0;
    keep(2 * M);
    CHECK(fake::blocks.count(p));
    fake::clock_shift += 2.0;
    DevBuf b;
    CHECK(b.alloc(64) == HISQ_OK && !fake::blocks.count(p) && fake::total == 2 * M + 64);
    fake::clock_shift += 6.0;
    b.recycle();
    CHECK(fake::total == 64);

    // a failing allocation takes everything that is kept
    p = keep(4 * M);
    fake::budget = 6 * M;
    CHECK(b.alloc(5 * M) == HISQ_OK && !fake::blocks.count(p) && fake::total == 5 * M);
    CHECK(hipGetLastError() == hipSuccess);
    fake::budget = ~(size_t)0;
    b.release();
    CHECK(fake::total == 0);

    // a block that the runtime does not free now is not lost
    keep(M);
    fake::free_fails = true;
    CHECK(hisq_release_memory(&freed) == HISQ_ERR_HIP && freed == 0);
    fake::clock_shift += 6.0;
    CHECK(b.alloc(64) == HISQ_OK && hipGetLastError() == hipSuccess);
    fake::free_fails = false;
    CHECK(hisq_release_memory(&freed) == HISQ_OK && freed == M);
    b.release();
    CHECK(fake::total == 0);
}

// Host memory that runs out in hisq_gauge_create is an error code, not an exception.
static size_t largest_new = ~(size_t)0;
void *operator new(size_t n) {
    void *p = n <= largest_new ? std::malloc(n) : nullptr;
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return n <= largest_new ? std::malloc(n) : nullptr; }
void *operator new[](size_t n) { return operator new(n); }
void *operator new[](size_t n, const std::nothrow_t &t) noexcept { return operator new(n, t); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }

static void create_without_host_memory() {
    const int dims[4] = {96, 96, 96, 24};
    const double *links = (const double *)0x10000;  // read by kernels only
    hisq_gauge_t g = nullptr;
    largest_new = 1 << 16;
    CHECK(hisq_gauge_create(&g, dims, links, links, HISQ_PREC_MASK(HISQ_PREC_FP32), nullptr) == HISQ_ERR_OOM && !g);
    CHECK(hisq_release_memory(nullptr) == HISQ_OK && fake::blocks.empty());
    largest_new = ~(size_t)0;
    CHECK(hisq_gauge_create(&g, dims, links, links, HISQ_PREC_MASK(HISQ_PREC_FP32), nullptr) == HISQ_OK);
    CHECK(hisq_gauge_destroy(g) == HISQ_OK);
}

// The autotuner times the default shape of every number of right-hand sides: where
// no launch is faster than the default's, that is what it installs.
static dim3 want_grid, want_block;
static void tuner_times_the_default() {
    const double *links = (const double *)0x10000;  // read by kernels only
    fake::launch_ms = [](dim3 g, dim3 b) {
        return g.x == want_grid.x && g.y == want_grid.y && b.x == want_block.x ? 0.5f : 1.f;
    };
    for (auto &dims : {std::array<int, 4>{8, 8, 8, 8}, {24, 24, 24, 8}, {32, 32, 32, 8}, {48, 48, 48, 12}, {28, 22, 18, 10}}) {
        hisq_gauge_t g = nullptr;
        CHECK(hisq_gauge_create(&g, dims.data(), links, links, HISQ_PREC_MASK_ALL, nullptr) == HISQ_OK);
        for (int prec : {HISQ_PREC_FP64, HISQ_PREC_FP32, HISQ_PREC_FP16S})
            for (int n = 1; n <= 17; ++n) {
                void *in = (void *)((uintptr_t)1 << 40), *out = (void *)((uintptr_t)1 << 41);
                int first[3], now[3];
                CHECK(hisq_dslash_shape(g, prec, n, 0, first) == HISQ_OK);
                CHECK(hisq_dslash_multi_rhs(g, 0, prec, n, in, out, nullptr, nullptr, nullptr) == HISQ_OK);
                want_grid = fake::last_grid;
                want_block = fake::last_block;
                CHECK(hisq_autotune(g, prec, n, nullptr, nullptr) == HISQ_OK);
                CHECK(hisq_dslash_shape(g, prec, n, 0, now) == HISQ_OK);
                CHECK(hisq_dslash_multi_rhs(g, 0, prec, n, in, out, nullptr, nullptr, nullptr) == HISQ_OK);
                if (fake::last_grid.x != want_grid.x || fake::last_grid.y != want_grid.y ||
                    fake::last_block.x != want_block.x) {
                    std::printf("FAILED %dx%dx%dx%d prec %d n %d: default (%d, %d, %#x), tuned (%d, %d, %#x)\n", dims[0],
                                dims[1], dims[2], dims[3], prec, n, first[0], first[1], first[2], now[0], now[1], now[2]);
                    std::exit(1);
                }
            }
        CHECK(hisq_gauge_destroy(g) == HISQ_OK && hisq_release_memory(nullptr) == HISQ_OK);
    }
}

// Default shapes of two right-hand sides on both sides of every limit.
static void two_rhs_shapes() {
    const double *links = (const double *)0x10000;  // read by kernels only
    const int SH = shared_order(2);
    const struct {
        std::array<int, 4> dims;
        int prec, tile, block, order;
    } want[] = {{{32, 32, 32, 8}, HISQ_PREC_FP64, 2, 256, 0},   {{48, 32, 24, 8}, HISQ_PREC_FP64, 2, 64, 0},
                {{32, 32, 16, 8}, HISQ_PREC_FP64, 1, 128, SH},  {{48, 48, 32, 12}, HISQ_PREC_FP64, 1, 128, SH},
                {{28, 28, 28, 8}, HISQ_PREC_FP64, 1, 128, SH},  {{24, 24, 24, 8}, HISQ_PREC_FP32, 1, 128, SH},
                {{32, 32, 32, 8}, HISQ_PREC_FP32, 2, 64, 0},    {{40, 40, 40, 8}, HISQ_PREC_FP32, 2, 256, 0},
                {{40, 40, 40, 8}, HISQ_PREC_FP16S, 2, 256, 0},  {{40, 40, 40, 8}, HISQ_PREC_FP16L, 1, 128, SH},
                {{48, 48, 48, 12}, HISQ_PREC_FP16L, 1, 128, SH}};
    for (auto &w : want) {
        hisq_gauge_t g = nullptr;
        CHECK(hisq_gauge_create(&g, w.dims.data(), links, links, HISQ_PREC_MASK_ALL, nullptr) == HISQ_OK);
        int s[3];
        for (int epi = 0; epi < 2; ++epi) {
            CHECK(hisq_dslash_shape(g, w.prec, 2, epi, s) == HISQ_OK);
            if (s[0] != w.tile || s[1] != w.block || s[2] != w.order) {
                std::printf("FAILED %dx%dx%dx%d prec %d: (%d, %d, %#x)\n", w.dims[0], w.dims[1], w.dims[2], w.dims[3],
                            w.prec, s[0], s[1], s[2]);
                std::exit(1);
            }
        }
        CHECK(hisq_gauge_destroy(g) == HISQ_OK && hisq_release_memory(nullptr) == HISQ_OK);
    }
}

int main(int argc, char **argv) {
    const std::string c = argc > 1 ? argv[1] : "";
    if (c == "destroy_other_device") destroy_other_device();
    else if (c == "training_without_memory") training_without_memory();
    else if (c == "create_without_host_memory") create_without_host_memory();
    else if (c == "tuner_times_the_default") tuner_times_the_default();
    else if (c == "two_rhs_shapes") two_rhs_shapes();
    else if (c == "network_blocks") network_blocks();
    else if (c == "destroy_while_refused") destroy_while_refused();
    else if (c == "kept_blocks") kept_blocks();
    else if (c == "failed_allocation") failed_allocation();
    else CHECK(!"a known case");
    std::printf("ok\n");
    return 0;
}
