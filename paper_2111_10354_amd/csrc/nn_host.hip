// Host orchestration of the preconditioner network: creation, weight I/O,
// forward application, loss and gradient over a batch of (A v, v) pairs by
// back-propagation through the adjoint layers, and Adam steps.

#include <algorithm>
#include <atomic>
#include <cstring>
#include <utility>

#include "nn_internal.h"

namespace hisq {

static NnGeom nn_geom(const hisq_gauge_s *g) {
    NnGeom G;
    for (int i = 0; i < 4; ++i) G.L[i] = g->dims[i];
    G.V = 2 * g->geom.vh;
    return G;
}

// layer input modes: the first layer (and the adjoint of the last) reads the
// one-channel even-site spinor, every other layer a hidden activation
enum { MODE_HIDDEN = 0, MODE_EVEN = 1 };

// Device buffers for `cap` training samples side by side, in one block: a new
// network's first step pays for every allocation.  The buffers that the network
// has are given up only for others: training goes on where these cannot be had.
static int train_alloc(hisq_nn_s *n, int cap) {
    const NnGeom G = nn_geom(n->gauge);
    const size_t act = nn_act_bytes(G), sb = spinor_bytes(F32, G.V / 2);
    hisq_nn_s::Train &t = n->train;
    const std::pair<hisq_nn_s::Train::Part *, size_t> parts[] = {
        {&t.act, std::max<size_t>((n->nlayers - 1) * act * cap, 16)},
        {&t.gbuf, 2 * act * cap},
        {&t.out, sb * cap},
        {&t.gout, sb * cap},
        {&t.partial, nn_wgrad_partial_floats(G) * 4 * cap},
        {&t.red, n->nweights * 8 * cap},
        {&t.scal, 8 * sizeof(double) * cap},
        {&t.partd, sizeof(double) * ((G.V / 2 + 255) / 256 + 1) * cap}};
    auto padded = [](size_t bytes) { return (bytes + 255) & ~(size_t)255; };
    size_t all = 0;
    for (auto &p : parts) all += padded(p.second);
    DevBuf mem;
    const int rc = mem.alloc(all);
    if (rc) return rc;
    t.mem.swap(mem);
    char *at = (char *)t.mem.p;
    for (auto &p : parts) {
        p.first->p = at;
        at += padded(p.second);
    }
    t.cap = cap;
    return HISQ_OK;
}

// Makes room for groups of `want` samples, or of as many as memory allows: half
// as many after each refusal.  A batch that memory did not suffice for, or a
// larger one, does not ask again.
static int train_reserve(hisq_nn_s *n, int want) {
    hisq_nn_s::Train &t = n->train;
    if (want <= t.cap || want >= t.refused) return HISQ_OK;
    for (int m = want; m > t.cap; m /= 2) {
        const int rc = train_alloc(n, m);
        if (rc != HISQ_ERR_OOM) return rc;
        t.refused = want;
    }
    return HISQ_OK;
}

// Samples that go through the layers together: all of the batch, within 512 MiB
// of buffers.  A sample's layer on 16^3 x 8 has one wavefront per SIMD and its
// reductions are 13 launches: 8 samples one by one 1.12 ms.  From 32^3 x 8 on
// one sample fills the card and the limit (4 samples there) costs nothing.
static int train_group(const hisq_nn_s *n, int batch) {
    const NnGeom G = nn_geom(n->gauge);
    const size_t one = (size_t)(n->nlayers + 1) * nn_act_bytes(G) + 2 * spinor_bytes(F32, G.V / 2) +
                       nn_wgrad_partial_floats(G) * 4;
    return (int)std::max<size_t>(1, std::min<size_t>(batch, ((size_t)512 << 20) / one));
}

int nn_create(hisq_nn_s **out, hisq_gauge_s *g, int nlayers, const int *ch, const double *weights, hipStream_t s) {
    static std::atomic<unsigned long long> next_id{1};
    hisq_nn_s *n = new (std::nothrow) hisq_nn_s();
    if (!n) {
        set_error("network: host allocation failed");
        return HISQ_ERR_OOM;
    }
    n->id = next_id++;
    n->gauge = g;
    n->nlayers = nlayers;
    n->ch.assign(ch, ch + nlayers + 1);
    const NnGeom G = nn_geom(g);
    size_t off = 0, aoff = 0, aoff_t = 0;
    std::vector<size_t> aoff_tv;
    for (int l = 0; l < nlayers; ++l) {
        n->woff.push_back(off);
        off += 2 * 9 * (size_t)ch[l] * ch[l + 1];
        n->aoff.push_back(aoff);
        aoff += nn_amat_elems(l == 0 ? MODE_EVEN : MODE_HIDDEN);
        aoff_tv.push_back(aoff_t);
        aoff_t += nn_amat_elems(l == nlayers - 1 ? MODE_EVEN : MODE_HIDDEN);
    }
    const size_t act = (size_t)(nlayers - 1) * nn_act_bytes(G);
    n->aoff.insert(n->aoff.end(), aoff_tv.begin(), aoff_tv.end());  // [fwd offsets..., adjoint offsets...]
    n->nweights = off;
    int rc;
    if ((rc = n->w.alloc(off * 8)) || (rc = n->m.alloc(off * 8)) || (rc = n->v.alloc(off * 8)) ||
        (rc = n->g.alloc(off * 8)) || (rc = n->amat.alloc(aoff * 2)) || (rc = n->amat_t.alloc(aoff_t * 2)) ||
        (rc = n->act.alloc(std::max<size_t>(act, 16))) || (rc = n->scal.alloc(8 * sizeof(double))) ||
        (rc = train_alloc(n, 1))) {
        delete n;
        return rc;
    }
    std::vector<double> zero(off, 0.0);
    HISQ_HIP_CHECK(hipMemcpyAsync(n->m.p, zero.data(), off * 8, hipMemcpyHostToDevice, s));
    HISQ_HIP_CHECK(hipMemcpyAsync(n->v.p, zero.data(), off * 8, hipMemcpyHostToDevice, s));
    HISQ_HIP_CHECK(hipMemcpyAsync(n->w.p, weights ? weights : zero.data(), off * 8, hipMemcpyHostToDevice, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    *out = n;
    return HISQ_OK;
}

static void build_amats(hisq_nn_s *n, hipStream_t s) {
    const int L = n->nlayers;
    for (int l = 0; l < L; ++l) {
        const double *W = (const double *)n->w.p + n->woff[l];
        nn_build_amat(W, n->ch[l], n->ch[l + 1], false, l == 0 ? MODE_EVEN : MODE_HIDDEN,
                      (__bf16 *)n->amat.p + n->aoff[l], s);
        nn_build_amat(W, n->ch[l], n->ch[l + 1], true, l == L - 1 ? MODE_EVEN : MODE_HIDDEN,
                      (__bf16 *)n->amat_t.p + n->aoff[L + l], s);
    }
    n->amat_valid = true;
}

static void *act_of(hisq_nn_s *n, int l) {  // output of layer l-1 = input of layer l (l >= 1)
    return (char *)n->act.p + (size_t)(l - 1) * nn_act_bytes(nn_geom(n->gauge));
}

// z = N(r): r and z even FP32 spinors (public layout)
int nn_forward(hisq_nn_s *n, const float *in, float *out, hipStream_t s) {
    hisq_gauge_s *g = n->gauge;
    if (!g->thin.p) {
        set_error("the gauge handle has no thin links (hisq_gauge_set_thin)");
        return HISQ_ERR_UNSUPPORTED;
    }
    if (!n->amat_valid) build_amats(n, s);
    const NnGeom G = nn_geom(g);
    const int L = n->nlayers;
    int rc;
    for (int l = 0; l < L; ++l) {
        const void *src = l == 0 ? (const void *)in : act_of(n, l);
        void *dst = l == L - 1 ? (void *)out : act_of(n, l + 1);
        const int inm = l == 0 ? MODE_EVEN : MODE_HIDDEN, outm = l == L - 1 ? MODE_EVEN : MODE_HIDDEN;
        if ((rc = nn_layer(G, g->thin.p, inm, outm, src, dst, (const __bf16 *)n->amat.p + n->aoff[l], 1, 0, 0, s)))
            return rc;
    }
    return HISQ_OK;
}

// Loss over a batch and its gradient, accumulated into n->g (overwritten);
// the loss ends in scal[3].  The samples go through the layers in groups; each
// sample's sums are its own, and samples are added in order, so the result
// does not depend on the grouping.
int nn_loss_grad_batch(hisq_nn_s *n, int batch, const float *av, const float *v, hipStream_t s) {
    hisq_gauge_s *g = n->gauge;
    const NnGeom G = nn_geom(g);
    const int vh = G.V / 2, L = n->nlayers;
    const size_t sb = spinor_bytes(F32, vh), act = nn_act_bytes(G);
    int rc;
    if ((rc = train_reserve(n, train_group(n, batch)))) return rc;
    HISQ_HIP_CHECK(hipMemsetAsync(n->g.p, 0, n->nweights * 8, s));
    HISQ_HIP_CHECK(hipMemsetAsync(n->scal.p, 0, 8 * sizeof(double), s));
    if (!n->amat_valid) build_amats(n, s);
    hisq_nn_s::Train &t = n->train;
    for (int first = 0; first < batch; first += t.cap) {
        const int m = std::min(t.cap, batch - first);
        const float *avi = (const float *)((const char *)av + sb * first);
        const float *vi = (const float *)((const char *)v + sb * first);
        auto hidden = [&](int l) { return (char *)t.act.p + (size_t)(l - 1) * t.cap * act; };  // input of layer l
        for (int l = 0; l < L; ++l) {
            const bool first_l = l == 0, last_l = l == L - 1;
            if ((rc = nn_layer(G, g->thin.p, first_l ? MODE_EVEN : MODE_HIDDEN, last_l ? MODE_EVEN : MODE_HIDDEN,
                               first_l ? (const void *)avi : hidden(l), last_l ? t.out.p : (void *)hidden(l + 1),
                               (const __bf16 *)n->amat.p + n->aoff[l], m, first_l ? sb : act, last_l ? sb : act, s)))
                return rc;
        }
        nn_loss_grad(vh, m, (const float *)t.out.p, vi, (float *)t.gout.p, (double *)t.partd.p, (double *)t.scal.p,
                     batch, s);
        void *gb[2] = {t.gbuf.p, (char *)t.gbuf.p + act * t.cap};
        const void *gcur = t.gout.p;
        int gmode = MODE_EVEN;
        for (int l = L - 1; l >= 0; --l) {
            const void *inl = l == 0 ? (const void *)avi : hidden(l);
            const int inm = l == 0 ? MODE_EVEN : MODE_HIDDEN;
            const size_t gstep = gmode == MODE_EVEN ? sb : act;
            if ((rc = nn_wgrad(G, g->thin.p, n->ch[l], n->ch[l + 1], inm, gmode, inl, gcur, m, l == 0 ? sb : act, gstep,
                               (float *)t.partial.p, (double *)t.red.p + n->woff[l], n->nweights, s)))
                return rc;
            if (l > 0) {
                void *gn = gb[l & 1];
                if ((rc = nn_layer(G, g->thin.p, gmode, MODE_HIDDEN, gcur, gn,
                                   (const __bf16 *)n->amat_t.p + n->aoff[L + l], m, gstep, act, s)))
                    return rc;
                gcur = gn;
                gmode = MODE_HIDDEN;
            }
        }
        nn_grad_add((const double *)t.red.p, (int)n->nweights, m, (double *)n->g.p, (const double *)t.scal.p,
                    (double *)n->scal.p + 3, s);
        HISQ_HIP_CHECK(hipGetLastError());
    }
    return HISQ_OK;
}

}  // namespace hisq

using namespace hisq;

static int nfail(int code, const char *msg) {
    set_error(msg);
    return code;
}

extern "C" {

int hisq_gauge_set_thin(hisq_gauge_t g, const double *thin, void *stream) {
    if (!g || !thin) return nfail(HISQ_ERR_INVALID, "gauge and thin links are required");
    std::lock_guard<std::mutex> lk(g->mu);
    const NnGeom G = nn_geom(g);
    int rc = g->thin.alloc(nn_thin_bytes(G));
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    if ((rc = nn_pack_thin(G, thin, g->thin.p, s))) return rc;
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    return HISQ_OK;
}

int hisq_nn_create(hisq_nn_t *out, hisq_gauge_t g, int nlayers, const int *channels, const double *weights,
                   void *stream) {
    if (!out || !g || !channels) return nfail(HISQ_ERR_INVALID, "out, gauge and channels are required");
    *out = nullptr;
    if (nlayers < 1 || nlayers > 8) return nfail(HISQ_ERR_INVALID, "1 <= nlayers <= 8");
    if (channels[0] != 1 || channels[nlayers] != 1)
        return nfail(HISQ_ERR_INVALID, "the first and last channel counts must be 1");
    for (int l = 0; l <= nlayers; ++l)
        if (!nn_channels_supported(channels[l])) return nfail(HISQ_ERR_UNSUPPORTED, "channel counts must be in 1..8");
    std::lock_guard<std::mutex> lk(g->mu);
    return nn_create(out, g, nlayers, channels, weights, (hipStream_t)stream);
}

int hisq_nn_destroy(hisq_nn_t net) {
    if (!net) return HISQ_OK;
    const OnDevice on(net->w.device);
    if (on.idle()) net->recycle();
    delete net;
    return HISQ_OK;
}

int hisq_nn_num_weights(hisq_nn_t net, size_t *n_complex) {
    if (!net || !n_complex) return nfail(HISQ_ERR_INVALID, "net and n_complex are required");
    *n_complex = net->nweights / 2;
    return HISQ_OK;
}

int hisq_nn_get_weights(hisq_nn_t net, double *weights, void *stream) {
    if (!net || !weights) return nfail(HISQ_ERR_INVALID, "net and weights are required");
    hipStream_t s = (hipStream_t)stream;
    HISQ_HIP_CHECK(hipMemcpyAsync(weights, net->w.p, net->nweights * 8, hipMemcpyDeviceToHost, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    return HISQ_OK;
}

int hisq_nn_set_weights(hisq_nn_t net, const double *weights, void *stream) {
    if (!net || !weights) return nfail(HISQ_ERR_INVALID, "net and weights are required");
    hipStream_t s = (hipStream_t)stream;
    HISQ_HIP_CHECK(hipMemcpyAsync(net->w.p, weights, net->nweights * 8, hipMemcpyHostToDevice, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    net->amat_valid = false;
    return HISQ_OK;
}

int hisq_nn_loss_grad(hisq_nn_t net, int batch, const void *av, const void *v, double *loss, double *grad,
                      void *stream) {
    TraceRange tr_("hisq_nn_loss_grad");
    if (!net || !av || !v || batch < 1) return nfail(HISQ_ERR_INVALID, "net, av, v and batch >= 1 are required");
    if (!net->gauge->thin.p) return nfail(HISQ_ERR_UNSUPPORTED, "the gauge handle has no thin links");
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lk(net->gauge->mu);
    int rc = nn_loss_grad_batch(net, batch, (const float *)av, (const float *)v, s);
    if (rc) return rc;
    double sc[8];
    HISQ_HIP_CHECK(hipMemcpyAsync(sc, net->scal.p, sizeof(sc), hipMemcpyDeviceToHost, s));
    if (grad) HISQ_HIP_CHECK(hipMemcpyAsync(grad, net->g.p, net->nweights * 8, hipMemcpyDeviceToHost, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    if (loss) *loss = sc[3];
    return HISQ_OK;
}

int hisq_nn_train_step(hisq_nn_t net, int batch, const void *av, const void *v, double lr, double *loss,
                       void *stream) {
    TraceRange tr_("hisq_nn_train_step");
    if (!net || !av || !v || batch < 1 || !(lr > 0.0))
        return nfail(HISQ_ERR_INVALID, "net, av, v, batch >= 1 and lr > 0 are required");
    if (!net->gauge->thin.p) return nfail(HISQ_ERR_UNSUPPORTED, "the gauge handle has no thin links");
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lk(net->gauge->mu);
    int rc = nn_loss_grad_batch(net, batch, (const float *)av, (const float *)v, s);
    if (rc) return rc;
    net->step += 1;
    nn_adam((double *)net->w.p, (double *)net->m.p, (double *)net->v.p, (const double *)net->g.p,
            (int)net->nweights, lr, net->step, s);
    net->amat_valid = false;
    double sc[8];
    HISQ_HIP_CHECK(hipMemcpyAsync(sc, net->scal.p, sizeof(sc), hipMemcpyDeviceToHost, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    if (loss) *loss = sc[3];
    return HISQ_OK;
}

int hisq_precond_apply(hisq_gauge_t g, hisq_nn_t net, const void *in, void *out, void *stream) {
    if (!g) return nfail(HISQ_ERR_INVALID, "gauge handle is NULL");
    if (!net || !in || !out) return nfail(HISQ_ERR_INVALID, "net, in and out are required");
    if (net->gauge != g) return nfail(HISQ_ERR_INVALID, "the network belongs to another gauge handle");
    if (in == out) return nfail(HISQ_ERR_INVALID, "in and out must not overlap");
    if (((uintptr_t)in & 15) || ((uintptr_t)out & 15)) return nfail(HISQ_ERR_INVALID, "buffers must be 16-byte aligned");
    std::lock_guard<std::mutex> lk(g->mu);
    return nn_forward(net, (const float *)in, (float *)out, (hipStream_t)stream);
}

}  // extern "C"
