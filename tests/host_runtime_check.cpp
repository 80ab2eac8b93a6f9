// Host code of libhisq.so against the stand-in runtime of host_runtime.h (no
// GPU).  usage: host_runtime_check CASE; prints "ok", or what failed.
#include "host_runtime.h"

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
    fake::max_block = 3 * have;  // a smaller batch may ask again
    CHECK(hisq_nn_loss_grad(net, 3, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
    CHECK(net->train.cap >= 2);
    const size_t grown = net->train.mem.bytes;
    fake::max_block = 0;  // nothing: the buffers stay
    CHECK(hisq_nn_loss_grad(net, 8, v.data(), v.data(), &loss, nullptr, nullptr) == HISQ_OK);
    CHECK(net->train.mem.bytes == grown);
    fake::max_block = ~(size_t)0;
    CHECK(hisq_nn_destroy(net) == HISQ_OK && hisq_gauge_destroy(g) == HISQ_OK);
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

int main(int argc, char **argv) {
    const std::string c = argc > 1 ? argv[1] : "";
    if (c == "destroy_other_device") destroy_other_device();
    else if (c == "training_without_memory") training_without_memory();
    else if (c == "failed_allocation") failed_allocation();
    else CHECK(!"a known case");
    std::printf("ok\n");
    return 0;
}
