// Gauge-covariant preconditioner network: forward, backward and Adam kernels.
//
// Layer with C_in -> C_out complex channels (C <= 8) on the full lattice:
//   y_a(x) = sum_b [ W0_ab psi_b(x) + sum_mu ( Wf_mu,ab U_mu(x) psi_b(x+mu)
//                                            + Wb_mu,ab U_mu(x-mu)^+ psi_b(x-mu) ) ]
// (linear, gauge covariant; the L-CNN construction of Favoni et al. 2022 used
// as a solver preconditioner as in Lehner and Wettig 2023).
//
// Storage in HBM:
//  * hidden activations and back-propagated gradients: BF16, always 8
//    channels (unused ones hold zeros).  A site is six 16-byte units
//    u = 2 colour + (0: re, 1: im), each holding channels 0..7, tiled by 64
//    sites: unit u of site s at byte ((s / 64) * 6 + u) * 1024 + (s % 64) * 16.
//  * network input and output: FP32 spinors of the public layout, even sites.
//  * thin links: FP16, a 144-byte record per site (links mu = 0..3 of 9
//    complex entries, entry k of link mu in 32-bit word 9 mu + k), tiled by 64
//    sites like the activations, nine units per site.
//
// Kernel: a wavefront owns 32 sites, i.e. 96 (site, colour) columns, and
// builds the layer as the real-block GEMM
//   [Re y; Im y] (16 x 96) = A (16 x K) B (K x 96),  A = [[Wr, -Wi], [Wi, Wr]],
// on v_mfma_f32_16x16x32_bf16 with FP32 accumulation.  B is the transported
// input, produced 32 K rows at a time (two paths x {re, im} x 8 channels) by
// the wave's lanes in FP32 and staged in LDS as BF16: lane pair (site, half)
// loads the neighbour's units and the link once per pair and each half
// transports 4 of the 8 channels.  The result is staged in LDS and written
// as whole 16-byte units.  The loads of a path are issued before the one ahead of
// it is transported, and a wavefront shares no LDS with another, so none waits
// for another.  The adjoint layer needed by back-propagation is
// the same kernel with weights W'_{p'} = W_p^H, p' the adjoint hop.  Weight
// gradients G(W_p[a][b]) = sum_{x,c} g_a(x)_c conj((T_p psi_b)(x)_c) use the
// same MFMA with (site, colour, re/im) as the reduction, per-block partials
// and a fixed-order final sum (deterministic).
//
// What bounds it (8 -> 8 channels, 32^3 x 8: 88 MB of links and activations, 12 us
// at 7.3 TB/s; 302 MB of neighbours from the L2s, 9 us; 1.2 GFLOP of transport,
// FP32 on the vector ALUs, which with its conversions and addresses is about 1700
// instructions per wavefront, 23 us): the vector ALUs, 41 us, 51 us with a
// path's loads issued when it was due and a barrier around every chunk.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "nn_internal.h"

namespace hisq {

typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef __bf16 b4v __attribute__((ext_vector_type(4)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s4v lds_s4v;

template <class T>
__device__ __forceinline__ cx<T> cconj(cx<T> a) { return {a.re, -a.im}; }

constexpr int NW_SITES = 32;                 // sites per wavefront
constexpr int NW_COLS = 3 * NW_SITES;        // (site, colour) columns per wavefront
constexpr int NN_WAVES = 2;                  // wavefronts per block
constexpr int NB_SITES = NW_SITES * NN_WAVES;
constexpr int BT_LD = 40;                    // bf16 per LDS column of B: 32 K rows + pad
constexpr int GT_LD = 2 * NW_COLS + 8;       // bf16 per LDS row of the gradient operand

enum { IO_FULL = 0, IO_EVEN = 1 };

// K extent of the real-block weight matrix: 9 paths x {re, im} x 8 channels
// padded to 160 for hidden inputs, 9 paths x {re, im} padded to 32 for the
// one-channel even-site input.
__host__ __device__ constexpr int kp_of(int inm) { return inm == IO_EVEN ? 32 : 160; }

// ------------------------------------------------------------------ geometry (full lattice, lex order)
struct Lex {
    int L[4];
    int V;
};

struct SiteGeo {
    int s;     // lex index
    int c[4];  // coordinates
    int par;   // (x + y + z + t) & 1
};

__device__ __forceinline__ SiteGeo site_geo(const Lex &g, int s) {
    SiteGeo o;
    o.s = s;
    int r = s;
    o.c[0] = r % g.L[0];
    r /= g.L[0];
    o.c[1] = r % g.L[1];
    r /= g.L[1];
    o.c[2] = r % g.L[2];
    o.c[3] = r / g.L[2];
    o.par = (o.c[0] + o.c[1] + o.c[2] + o.c[3]) & 1;
    return o;
}

// Step of the lex index from coordinate c of an axis of extent L to c + d, d = +1
// or -1.  A choice of two numbers, no branch: a branch ends the block in which the
// loads of the paths are scheduled.
__device__ __forceinline__ int hop_step(int c, int L, int stride, int d) {
    const int wrap = (L - 1) * stride;
    return c == (d > 0 ? L - 1 : 0) ? -d * wrap : d * stride;
}

// lex index of x + d mu
template <int MU>
__device__ __forceinline__ int hop(const Lex &g, const SiteGeo &x, int d) {
    int stride = 1;
#pragma unroll
    for (int k = 0; k < MU; ++k) stride *= g.L[k];
    return x.s + hop_step(x.c[MU], g.L[MU], stride, d);
}

// Enumerated site -> lex index: all sites in lex order, or the even sites in
// checkerboard order (h = lex / 2).
template <int MODE>
__device__ __forceinline__ int site_of(const Lex &g, int idx) {
    if constexpr (MODE == IO_FULL) {
        return idx;
    } else {
        const int lxh = g.L[0] >> 1;
        const int xh = idx % lxh, r = idx / lxh;
        const int y = r % g.L[1], z = (r / g.L[1]) % g.L[2], t = r / (g.L[1] * g.L[2]);
        return 2 * xh + ((y + z + t) & 1) + g.L[0] * (y + g.L[1] * (z + g.L[2] * t));
    }
}

// ------------------------------------------------------------------ thin links (FP16)
// The words of link mu of site s: from word mu of unit 2 mu of the record on.
// Only those are loaded: a register of an unused word is given to another value
// while the load is in flight, which then waits for it.
template <int MU>
__device__ __forceinline__ void load_link(const void *thin, int s, unsigned wd[9]) {
    const unsigned *b = (const unsigned *)thin + ((size_t)(s >> 6) * 9 * 64 + (s & 63) + 2 * MU * 64) * 4;
#pragma unroll
    for (int k = 0; k < 9; ++k) wd[k] = b[(MU + k) / 4 * 256 + (MU + k) % 4];
}

// The same for a mu that differs from lane to lane
__device__ __forceinline__ void load_link(const void *thin, int s, int mu, unsigned wd[9]) {
    const u4v *b = (const u4v *)thin + (size_t)(s >> 6) * 9 * 64 + (s & 63) + 2 * mu * 64;
    const u4v r[3] = {b[0], b[64], b[128]};
    unsigned w[12] = {r[0].x, r[0].y, r[0].z, r[0].w, r[1].x, r[1].y, r[1].z, r[1].w, r[2].x, r[2].y, r[2].z, r[2].w};
    // words from mu on, in two shifts with masks: a choice of elements would put
    // the array into scratch memory
    const unsigned m1 = 0u - (mu & 1), m2 = 0u - ((mu >> 1) & 1);
#pragma unroll
    for (int k = 0; k < 11; ++k) w[k] = (w[k] & ~m1) | (w[k + 1] & m1);
#pragma unroll
    for (int k = 0; k < 9; ++k) wd[k] = (w[k] & ~m2) | (w[k + 2] & m2);
}

__device__ __forceinline__ void unpack_link(const unsigned wd[9], cx<float> w[9]) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const unsigned v = wd[k];
        const h2v h = __builtin_bit_cast(h2v, v);
        w[k] = {(float)h.x, (float)h.y};
    }
}

// Pack canonical FP64 thin links [V][4][3][3] complex into the FP16 records;
// *bad is set if an entry is not finite or too large for FP16.
__global__ __launch_bounds__(256) void k_pack_thin(Lex g, const double *__restrict__ U, void *dst, unsigned *bad) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int mu = blockIdx.y;
    if (s >= g.V) return;
    unsigned *words = (unsigned *)dst;
    const double *src = U + ((size_t)s * 4 + mu) * 18;
    bool ok = true;
    for (int k = 0; k < 9; ++k) {
        const int wi = 9 * mu + k, e = wi >> 2, q = wi & 3;
        const double re = src[2 * k], im = src[2 * k + 1];
        ok = ok && fabs(re) < 32768.0 && fabs(im) < 32768.0;  // false for NaN as well
        const h2v h = {(_Float16)(float)re, (_Float16)(float)im};
        words[((size_t)(s >> 6) * 9 + e) * 256 + (size_t)(s & 63) * 4 + q] = __builtin_bit_cast(unsigned, h);
    }
    if (!ok) atomicOr(bad, 1u);
}

// ------------------------------------------------------------------ activations
__device__ __forceinline__ float bf_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

// Channels 4 h .. 4 h + 3 of the six units of site s: v[u] = 8 bytes of unit u.
__device__ __forceinline__ void load_act_half(const void *buf, int s, int h, u2v v[6]) {
    const u2v *b = (const u2v *)buf + ((size_t)(s >> 6) * 6 * 64 + (s & 63)) * 2 + h;
#pragma unroll
    for (int u = 0; u < 6; ++u) v[u] = b[(size_t)u * 128];
}

// channel q (0..3) of an 8-byte half unit
__device__ __forceinline__ float half_chan(const u2v &v, int q) {
    const unsigned w = (q < 2) ? v.x : v.y;
    return (q & 1) ? bf_hi(w) : bf_lo(w);
}

// ------------------------------------------------------------------ transport into LDS
// A wavefront writes and reads its own part of the LDS, whose accesses of one
// wavefront stay in order: the compiler has to keep their order, nothing waits.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <class F, int... K>
__device__ __forceinline__ void for_paths(F &&f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K>{}), ...);
}

// What path P (0 identity, 1..4 forward hop mu = P - 1, 5..8 backward hop
// mu = P - 5) reads for channels 4h .. 4h + 3 of a hidden input at site x
struct PathData {
    unsigned link[9];
    u2v v[6];
};

template <int P>
__device__ __forceinline__ void load_path(const Lex &g, const void *thin, const void *in, const SiteGeo &x, int h,
                                          PathData &d) {
    int nb = x.s, ls = x.s;
    if constexpr (P >= 1 && P <= 4) nb = hop<P - 1>(g, x, +1);
    if constexpr (P >= 5) ls = nb = hop<P - 5>(g, x, -1);
    if constexpr (P >= 1) load_link<(P - 1) & 3>(thin, ls, d.link);
    load_act_half(in, nb, h, d.v);
}

// Transports them and writes the 3 colours x {re, im} x 4 channels to the LDS
// columns of the site at K offset koff (+ 8 ri + 4 h); P = 9 is padding.
template <int P>
__device__ __forceinline__ void transport_path(const PathData &d, int h, __bf16 *col, int koff) {
    float tr[3][4], ti[3][4];
    if constexpr (P == 9) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) tr[a][q] = ti[a][q] = 0.f;
    } else {
        cx<float> w[9];
        if constexpr (P >= 1) unpack_link(d.link, w);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cx<float> vb[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) vb[c] = {half_chan(d.v[2 * c], q), half_chan(d.v[2 * c + 1], q)};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                cx<float> t = {0.f, 0.f};
                if constexpr (P == 0) {
                    t = vb[a];
                } else if constexpr (P <= 4) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) cmac(t, w[3 * a + c], vb[c]);
                } else {
#pragma unroll
                    for (int c = 0; c < 3; ++c) cmac(t, cconj(w[3 * c + a]), vb[c]);  // conj(U[c][a]) v[c]
                }
                tr[a][q] = t.re;
                ti[a][q] = t.im;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const b4v r = {(__bf16)tr[a][0], (__bf16)tr[a][1], (__bf16)tr[a][2], (__bf16)tr[a][3]};
        const b4v i = {(__bf16)ti[a][0], (__bf16)ti[a][1], (__bf16)ti[a][2], (__bf16)ti[a][3]};
        *(b4v *)(col + a * BT_LD + koff + 4 * h) = r;
        *(b4v *)(col + a * BT_LD + koff + 8 + 4 * h) = i;
    }
}

// All paths of a hidden input, two to a chunk of 32 K rows: use(q) once chunk q
// is in LDS.  The loads of the next PATH_AHEAD paths are in flight; two of them
// take 21 registers more and the same time (41.1 against 40.6 us above).  A site
// past the last (valid false) is site 0, or zero if ZERO is set.
constexpr int PATH_AHEAD = 1;

template <bool ZERO, class F>
__device__ __forceinline__ void transport_hidden(const Lex &g, const void *thin, const void *in, const SiteGeo &x,
                                                 bool valid, int h, __bf16 *col, F &&use) {
    PathData d[PATH_AHEAD + 1];
    for_paths([&](auto pc) { load_path<decltype(pc)::value>(g, thin, in, x, h, d[decltype(pc)::value]); },
              std::make_integer_sequence<int, PATH_AHEAD>{});
    auto path = [&](auto pc) {
        constexpr int P = decltype(pc)::value, N = P + PATH_AHEAD, S = P % (PATH_AHEAD + 1);
        if constexpr (N <= 8) load_path<N>(g, thin, in, x, h, d[N % (PATH_AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ZERO) {
#pragma unroll
            for (int u = 0; u < 6; ++u) d[S].v[u] = valid ? d[S].v[u] : u2v{0u, 0u};
        }
        transport_path<P>(d[S], h, col, (P & 1) * 16);
        if constexpr (P == 8) transport_path<9>(d[S], h, col, 16);
        if constexpr (P == 8 || (P & 1)) {
            wave_sync();
            use(std::integral_constant<int, P / 2>{});
            wave_sync();
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for_paths(path, std::make_integer_sequence<int, 9>{});
}

// The one-channel even-site input (FP32 public spinor): path p of a column at
// K = p KS and p KS + RI (re, im), all other rows zero.  It lives on the even
// sites, so path 0 reaches the even sites and the hops the odd ones: of a full
// lattice's enumeration each four lanes take two neighbours in x, one of either
// parity, and a lane the two hops of one direction (1 -> 8 channels, 32^3 x 8:
// 17.8 us; 20.2 us with every lane pair on all eight hops of its site).
template <int MODE, int KS, int RI>
__device__ __forceinline__ void transport_even(const Lex &g, const void *thin, const float *in, int base, int nsites,
                                               int l, __bf16 *bt) {
    const Spinor<F32> src{const_cast<float *>(in), g.V / 2};
    const u4v zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = l; e < NW_COLS * 4; e += 64) *(u4v *)(bt + (e >> 2) * BT_LD + (e & 3) * 8) = zero;
    wave_sync();
    auto put = [&](int s, int a, int p, const cx<float> &t) {
        __bf16 *c = bt + (3 * s + a) * BT_LD + p * KS;
        c[0] = (__bf16)t.re;
        c[RI] = (__bf16)t.im;
    };
    if constexpr (MODE == IO_EVEN) {
        if (l < NW_SITES && base + l < nsites) {
            cx<float> t[3];
            src.load(base + l, t);
#pragma unroll
            for (int a = 0; a < 3; ++a) put(l, a, 0, t[a]);
        }
    } else {
        const int pair = 2 * (l >> 2), mu = l & 3;
        if (base + pair < nsites) {  // V is a multiple of 16
            SiteGeo x = site_geo(g, base + pair);
            const int odd = x.par ? 0 : 1;
            cx<float> t0[3];
            src.load((base + pair) >> 1, t0);
            const cx<float> own = {mu == 0 ? +t0[0].re : mu == 1 ? +t0[1].re : +t0[2].re,
                                   mu == 0 ? +t0[0].im : mu == 1 ? +t0[1].im : +t0[2].im};
            if (mu < 3) put(pair + 1 - odd, mu, 0, own);
            x.s += odd;
            x.c[0] += odd;
            const int c = mu == 0 ? +x.c[0] : mu == 1 ? +x.c[1] : mu == 2 ? +x.c[2] : +x.c[3];
            const int Lm = mu == 0 ? +g.L[0] : mu == 1 ? +g.L[1] : mu == 2 ? +g.L[2] : +g.L[3];
            const int st = mu == 0 ? 1 : mu == 1 ? g.L[0] : g.L[0] * g.L[1] * (mu == 2 ? 1 : +g.L[2]);
            const int nf = x.s + hop_step(c, Lm, st, +1), nb = x.s + hop_step(c, Lm, st, -1);
            unsigned lf[9], lb[9];
            cx<float> vf[3], vb[3], w[9];
            load_link(thin, x.s, mu, lf);
            load_link(thin, nb, mu, lb);
            src.load(nf >> 1, vf);
            src.load(nb >> 1, vb);
            unpack_link(lf, w);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                cx<float> t = {0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 3; ++k) cmac(t, w[3 * a + k], vf[k]);
                put(pair + odd, a, 1 + mu, t);
            }
            unpack_link(lb, w);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                cx<float> t = {0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 3; ++k) cmac(t, cconj(w[3 * k + a]), vb[k]);
                put(pair + odd, a, 5 + mu, t);
            }
        }
    }
}

// ------------------------------------------------------------------ layer kernel
// amat: bf16 [16][kp_of(INM)], rows 0..7 Re and 8..15 Im of the output
// channels.  OUTM == IO_FULL: all V sites, output BF16 hidden units;
// IO_EVEN: even sites in checkerboard order, output channel 0 as an FP32
// public spinor.  One grid row per sample, `in` and `out` of sample y `in_step`
// and `out_step` bytes on from those of the sample before.
template <int INM, int OUTM>
__global__ __launch_bounds__(64 * NN_WAVES) void k_nn_layer(Lex g, const void *thin, const void *__restrict__ in0,
                                                            void *__restrict__ out0, const __bf16 *__restrict__ amat,
                                                            size_t in_step, size_t out_step) {
    constexpr int KP = kp_of(INM);
    const void *__restrict__ in = (const char *)in0 + in_step * blockIdx.y;
    void *__restrict__ out = (char *)out0 + out_step * blockIdx.y;
    __shared__ __attribute__((aligned(16))) __bf16 Bt[NN_WAVES][NW_COLS][BT_LD];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, j = l >> 4;
    const int nsites = OUTM == IO_FULL ? g.V : g.V / 2;
    const int base = (blockIdx.x * NN_WAVES + w) * NW_SITES;

    b8v am[KP / 32];
#pragma unroll
    for (int q = 0; q < KP / 32; ++q) am[q] = *(const b8v *)(amat + i * KP + q * 32 + j * 8);
    f4v acc[6];
#pragma unroll
    for (int cb = 0; cb < 6; ++cb) acc[cb] = f4v{0.f, 0.f, 0.f, 0.f};
    auto product = [&](auto qc) {
#pragma unroll
        for (int cb = 0; cb < 6; ++cb) {
            const b8v b = *(const b8v *)(&Bt[w][cb * 16 + i][j * 8]);
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[decltype(qc)::value], b, acc[cb], 0, 0, 0);
        }
    };
    if constexpr (INM == IO_EVEN) {
        transport_even<OUTM, 2, 1>(g, thin, (const float *)in, base, nsites, l, &Bt[w][0][0]);
        wave_sync();
        product(std::integral_constant<int, 0>{});
        wave_sync();
    } else {
        const int sl = l >> 1, h = l & 1;  // lane pair (site, half)
        const bool valid = base + sl < nsites;
        const SiteGeo x = site_geo(g, valid ? site_of<OUTM>(g, base + sl) : 0);
        transport_hidden<false>(g, thin, in, x, valid, h, &Bt[w][sl * 3][0], product);
    }

    // lane (i, j) holds rows 4j .. 4j + 3 of column cb * 16 + i
    if constexpr (OUTM == IO_FULL) {
        __bf16 *Ot = &Bt[w][0][0];  // staging [32 sites][48] (unit u = 2 colour + ri, channel)
#pragma unroll
        for (int cb = 0; cb < 6; ++cb) {
            const int cl = cb * 16 + i, s = cl / 3, c = cl % 3;
            const b4v v = {(__bf16)acc[cb][0], (__bf16)acc[cb][1], (__bf16)acc[cb][2], (__bf16)acc[cb][3]};
            *(b4v *)(Ot + s * 48 + (2 * c + (j >> 1)) * 8 + (j & 1) * 4) = v;
        }
        wave_sync();
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = t * 64 + l, s = e & 31, u = e >> 5;
            const int S = base + s;
            if (S < nsites) {
                const u4v val = *(const u4v *)(Ot + s * 48 + u * 8);
                ((u4v *)out)[((size_t)(S >> 6) * 6 + u) * 64 + (S & 63)] = val;
            }
        }
    } else {
        float *Of = (float *)&Bt[w][0][0];  // [32 sites][6]
#pragma unroll
        for (int cb = 0; cb < 6; ++cb) {
            const int cl = cb * 16 + i, s = cl / 3, c = cl % 3;
            if (j == 0) Of[s * 6 + 2 * c] = acc[cb][0];      // row 0: Re of channel 0
            if (j == 2) Of[s * 6 + 2 * c + 1] = acc[cb][0];  // row 8: Im of channel 0
        }
        wave_sync();
        if (l < NW_SITES && base + l < nsites) {
            cx<float> v[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] = {Of[l * 6 + 2 * c], Of[l * 6 + 2 * c + 1]};
            Spinor<F32>{(float *)out, g.V / 2}.store(base + l, v);
        }
    }
}

// ------------------------------------------------------------------ weight gradient
// Per block: partial[blk][16][KC], KC = 80 (hidden input: column 8 p + b) or
// 16 (even input: column p), C[r][n] = sum over the block's (site, colour) of
// r < 8: Re(g_r conj t_n), r >= 8: Im(g_{r-8} conj t_n).  The upstream gradient
// g has mode GM (IO_FULL: BF16 hidden units on all sites; IO_EVEN: channel 0
// as an FP32 public spinor on even sites); sites are enumerated like the
// layer kernel with OUTM = GM.  One grid row per sample, as in the layer kernel.
// Its reduction runs along the columns of the transported tile, across the rows
// in which LDS holds it: the transposing LDS read gives four columns at once,
// and the half of A2 that repeats the other is not stored (22 KB of LDS for 38).
// 8 samples of 16^3 x 8, 8 -> 8 channels 80.5 -> 40.4 us, 8 -> 1 46.7 -> 26.5,
// 1 -> 8 35.8 -> 16.0.
template <int INM, int GM>
__global__ __launch_bounds__(64 * NN_WAVES) void k_nn_wgrad(Lex g, const void *thin, const void *__restrict__ in0,
                                                            const void *__restrict__ grad0, float *__restrict__ partial,
                                                            size_t in_step, size_t grad_step) {
    const void *__restrict__ in = (const char *)in0 + in_step * blockIdx.y;
    const void *__restrict__ grad = (const char *)grad0 + grad_step * blockIdx.y;
    constexpr int KP = kp_of(INM);
    constexpr int NQ = KP / 32;  // chunks
    constexpr int KC = INM == IO_EVEN ? 16 : 80;
    constexpr int BT_B = NW_COLS * BT_LD, GT_B = 8 * GT_LD;  // bf16 of a wave's operands
    // the block's partial sums take the operands' place at the end
    constexpr int RED_LD = 20, WAVE_B = std::max(BT_B + GT_B, 2 * RED_LD * KC);
    __shared__ __attribute__((aligned(16))) __bf16 lds[NN_WAVES][WAVE_B];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, j = l >> 4;
    __bf16 *Bt = &lds[w][0], *Gt = Bt + BT_B;
    const int nsites = GM == IO_FULL ? g.V : g.V / 2;
    const int base = (blockIdx.x * NN_WAVES + w) * NW_SITES;

    // A2 = [[Gr, Gi], [Gi, -Gr]] over m = (site, colour): re block m < 96, im
    // block m >= 96.  Its upper half is kept; the lower is read from it.
    if constexpr (GM == IO_FULL) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = t * 64 + l, s = e & 31, u = e >> 5, c = u >> 1, ri = u & 1;
            const int S = base + s, m = s * 3 + c;
            u4v val = {0u, 0u, 0u, 0u};
            if (S < nsites) val = ((const u4v *)grad)[((size_t)(S >> 6) * 6 + u) * 64 + (S & 63)];
            const b8v v = __builtin_bit_cast(b8v, val);
#pragma unroll
            for (int a = 0; a < 8; ++a) Gt[a * GT_LD + ri * NW_COLS + m] = v[a];
        }
    } else {
        const u4v zero = {0u, 0u, 0u, 0u};
        for (int e = l; e < GT_B / 8; e += 64) ((u4v *)Gt)[e] = zero;
        wave_sync();
        if (l < NW_SITES) {
            cx<float> v[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
            if (base + l < nsites) Spinor<F32>{(float *)grad, g.V / 2}.load(base + l, v);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                Gt[l * 3 + c] = (__bf16)v[c].re;
                Gt[NW_COLS + l * 3 + c] = (__bf16)v[c].im;
            }
        }
    }

    f4v acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = f4v{0.f, 0.f, 0.f, 0.f};
    const __bf16 *grow = Gt + (i & 7) * GT_LD;
    const bool lower = i >= 8;
    auto product = [&](auto qc) {
#pragma unroll
        for (int ks = 0; ks < (2 * NW_COLS) / 32; ++ks) {
            const int ri = ks >= 3 ? 1 : 0;
            const int ga = ks * 32 + j * 8, gb = ga + (ri ? -NW_COLS : NW_COLS);
            u4v ar = *(const u4v *)(grow + (lower ? gb : ga));
            if (ri) ar ^= lower ? 0x80008000u : 0u;
            // columns m = (ks % 3) 32 + 8 j + 0..7 of the transported tile, row i
            // of its re or im block: the tile is transposed as it is read, each 16
            // lanes four columns of 16 rows at a time
            const int n = (i & 3) * 4;
            const __bf16 *src = Bt + ((ks % 3) * 32 + j * 8 + (i >> 2)) * BT_LD +
                                (INM == IO_EVEN ? ri * 16 + n : (n >> 3) * 16 + ri * 8 + (n & 7));
            const s4v b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)src);
            const s4v b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)(src + 4 * BT_LD));
            const s8v b = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
            acc[decltype(qc)::value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(b8v, ar), __builtin_bit_cast(b8v, b), acc[decltype(qc)::value], 0, 0, 0);
        }
    };
    if constexpr (INM == IO_EVEN) {
        transport_even<GM, 1, 16>(g, thin, (const float *)in, base, nsites, l, Bt);
        wave_sync();
        product(std::integral_constant<int, 0>{});
    } else {
        const int sl = l >> 1, h = l & 1;  // lane pair (site, half)
        const bool valid = base + sl < nsites;
        const SiteGeo x = site_geo(g, valid ? site_of<GM>(g, base + sl) : 0);
        transport_hidden<true>(g, thin, in, x, valid, h, Bt + sl * 3 * BT_LD, product);
    }
    wave_sync();
    // [KC][16 rows + pad]: a lane's four rows are one store
    float *Red = (float *)Bt;
#pragma unroll
    for (int q = 0; q < NQ; ++q) *(f4v *)(Red + (q * 16 + i) * RED_LD + j * 4) = acc[q];
    __syncthreads();
    // sum the block's waves in a fixed order, write the block partial
    for (int e = threadIdx.x; e < 16 * KC; e += blockDim.x) {
        const int r = e / KC, k = e % KC;
        float s = 0.f;
        for (int ww = 0; ww < NN_WAVES; ++ww) s += ((const float *)&lds[ww][0])[k * RED_LD + r];
        partial[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 16 * KC + e] = s;
    }
}

// Three-stage fixed-order sum of the block partials.  Stage 1: segment sg of
// sample z's blocks, every entry e of the 16 x KC partial: fold[z][sg][e].
constexpr int NN_FOLD = 64;  // segments

__global__ __launch_bounds__(256) void k_nn_wgrad_fold(const float *__restrict__ partial, int nblk, int nent,
                                                      float *__restrict__ fold) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x, sg = blockIdx.y;
    if (e >= nent) return;
    partial += (size_t)blockIdx.z * nblk * nent;
    const int per = (nblk + NN_FOLD - 1) / NN_FOLD;
    const int b0 = sg * per, b1 = min(nblk, b0 + per);
    float s = 0.f;
    for (int b = b0; b < b1; ++b) s += partial[(size_t)b * nent + e];
    fold[((size_t)blockIdx.z * NN_FOLD + sg) * nent + e] = s;
}

// Stage 2: the layer's part of sample y's gradient, [p][a][b] (complex double)
// = sum over the segments (fixed order); `step` doubles from sample to sample.
__global__ void k_nn_wgrad_reduce(const float *__restrict__ fold, int inm, int cin, int cout, double *red,
                                  size_t step) {
    const int KC = inm == IO_EVEN ? 16 : 80;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;  // (a, p, b)
    if (e >= cout * 9 * cin) return;
    const int a = e / (9 * cin), pb = e % (9 * cin), p = pb / cin, b = pb % cin;
    const int n = inm == IO_EVEN ? p : 8 * p + b;
    fold += (size_t)blockIdx.y * NN_FOLD * 16 * KC;
    double re = 0.0, im = 0.0;
#pragma unroll 16
    for (int sg = 0; sg < NN_FOLD; ++sg) {
        const float *P = fold + (size_t)sg * 16 * KC;
        re += P[a * KC + n];
        im += P[(8 + a) * KC + n];
    }
    double *gp = red + step * blockIdx.y + 2 * (((size_t)p * cout + a) * cin + b);
    gp[0] = re;
    gp[1] = im;
}

// Stage 3, all weights: grad += the samples' gradients, one after another;
// thread n adds the samples' losses (scal[8 z + 3]) to *loss the same way.
__global__ void k_nn_grad_add(const double *__restrict__ red, int n, int samples, double *__restrict__ grad,
                              const double *__restrict__ scal, double *loss) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        double s = grad[i];
        for (int z = 0; z < samples; ++z) s += red[(size_t)z * n + i];
        grad[i] = s;
    } else if (i == n) {
        double s = *loss;
        for (int z = 0; z < samples; ++z) s += scal[8 * z + 3];
        *loss = s;
    }
}

// Real-block bf16 matrix of a layer (transposed = the adjoint layer), in the
// K order of the input mode: hidden k = 16 p + 8 ri + b, even k = 2 p + ri.
__global__ void k_nn_build_amat(const double *__restrict__ W, int cin, int cout, int transposed, int inm,
                                __bf16 *amat) {
    // forward: out channels cout, in channels cin; transposed: out = cin, in = cout
    const int ci = transposed ? cout : cin, co = transposed ? cin : cout;
    const int KP = kp_of(inm);
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 16 * KP) return;
    const int r = e / KP, k = e % KP;
    int p, ri, b;
    if (inm == IO_EVEN) {
        p = k >> 1;
        ri = k & 1;
        b = 0;
    } else {
        p = k >> 4;
        ri = (k >> 3) & 1;
        b = k & 7;
    }
    double val = 0.0;
    const int a = r & 7;
    if (p < 9 && a < co && b < ci) {
        double wr, wi;
        if (!transposed) {  // y_a += W_p[a][b] t_{p,b}
            const double *src = W + 2 * (((size_t)p * cout + a) * cin + b);
            wr = src[0];
            wi = src[1];
        } else {  // W'_{p'}[a][b] = conj(W_p[b][a]), p' adjoint of p
            const int pf = p == 0 ? 0 : (p <= 4 ? p + 4 : p - 4);
            const double *src = W + 2 * (((size_t)pf * cout + b) * cin + a);
            wr = src[0];
            wi = -src[1];
        }
        const bool im_row = r >= 8, im_col = ri == 1;
        // [[Wr, -Wi], [Wi, Wr]]
        val = !im_row ? (!im_col ? wr : -wi) : (!im_col ? wi : wr);
    }
    amat[e] = (__bf16)(float)val;
}

// loss pieces on even sites, one grid row per sample: partial |out - v|^2 and
// G(out) = scale (out - v)
__global__ __launch_bounds__(256) void k_nn_loss_grad(Spinor<F32> out, Spinor<F32> v, const double *__restrict__ scal,
                                                      Spinor<F32> gout, double *__restrict__ part) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x, z = blockIdx.y;
    double dd = 0.0;
    if (h < v.vh) {
        cx<float> o[3], t[3], gg[3];
        out.rhs(z).load(h, o);
        v.rhs(z).load(h, t);
        const float sc = (float)scal[8 * z + 1];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float dr = o[c].re - t[c].re, di = o[c].im - t[c].im;
            dd += (double)dr * dr + (double)di * di;
            gg[c] = {sc * dr, sc * di};
        }
        gout.rhs(z).store(h, gg);
    }
    __shared__ double red[4];
    for (int off = 32; off >= 1; off >>= 1) dd += __shfl_xor(dd, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dd;
    __syncthreads();
    if (threadIdx.x == 0) part[(size_t)z * gridDim.x + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void k_nn_norm2(Spinor<F32> v, double *__restrict__ part) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x, z = blockIdx.y;
    double dd = 0.0;
    if (h < v.vh) {
        cx<float> t[3];
        v.rhs(z).load(h, t);
#pragma unroll
        for (int c = 0; c < 3; ++c) dd += (double)t[c].re * t[c].re + (double)t[c].im * t[c].im;
    }
    __shared__ double red[4];
    for (int off = 32; off >= 1; off >>= 1) dd += __shfl_xor(dd, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dd;
    __syncthreads();
    if (threadIdx.x == 0) part[(size_t)z * gridDim.x + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Sample z's scalars s = scal + 8 z from the sum of its n partials (fixed
// order); mode 0: scale = 2 / (B |v|^2) into s[1], keep |v|^2 in s[2];
// mode 1: its part of the loss, sum / (|v|^2 B), into s[3]
__global__ void k_nn_scalar(const double *__restrict__ part, int n, double *scal, int mode, int batch) {
    __shared__ double red[256];
    double *s = scal + 8 * blockIdx.x;
    part += (size_t)blockIdx.x * n;
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) acc += part[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < (int)blockDim.x; ++i) t += red[i];
        if (mode == 0) {
            s[2] = t;
            s[1] = t > 0.0 ? 2.0 / ((double)batch * t) : 0.0;
        } else {
            s[3] = s[2] > 0.0 ? t / (s[2] * (double)batch) : 0.0;
        }
    }
}

// Adam on the real and imaginary parts of every weight (FP64 master copy).
__global__ void k_nn_adam(double *w, double *m, double *v, const double *g, int n, double lr, double b1, double b2,
                          double eps, int step) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double gi = g[i];
    m[i] = b1 * m[i] + (1.0 - b1) * gi;
    v[i] = b2 * v[i] + (1.0 - b2) * gi * gi;
    const double mh = m[i] / (1.0 - pow(b1, (double)step));
    const double vh = v[i] / (1.0 - pow(b2, (double)step));
    w[i] -= lr * mh / (sqrt(vh) + eps);
}

// ------------------------------------------------------------------ dispatch
static Lex lex_of(const NnGeom &G) { return Lex{{G.L[0], G.L[1], G.L[2], G.L[3]}, G.V}; }

static int grid_blocks(int nsites) { return (nsites + NB_SITES - 1) / NB_SITES; }

bool nn_channels_supported(int c) { return c >= 1 && c <= 8; }

size_t nn_act_bytes(const NnGeom &G) { return (size_t)((G.V + 63) / 64) * 6 * 1024; }

size_t nn_amat_elems(int inm) { return (size_t)16 * kp_of(inm); }

size_t nn_wgrad_partial_floats(const NnGeom &G) { return ((size_t)grid_blocks(G.V) + NN_FOLD) * 16 * 80; }

size_t nn_thin_bytes(const NnGeom &G) { return (size_t)((G.V + 63) / 64) * 9 * 1024 + 256; }

int nn_layer(const NnGeom &G, const void *thin, int inm, int outm, const void *in, void *out, const void *amat,
             int samples, size_t in_step, size_t out_step, hipStream_t s) {
    const Lex L = lex_of(G);
    const dim3 grid(grid_blocks(outm == IO_FULL ? G.V : G.V / 2), samples), block(64 * NN_WAVES);
    const __bf16 *A = (const __bf16 *)amat;
    if (inm == IO_FULL && outm == IO_FULL)
        hipLaunchKernelGGL((k_nn_layer<IO_FULL, IO_FULL>), grid, block, 0, s, L, thin, in, out, A, in_step, out_step);
    else if (inm == IO_EVEN && outm == IO_FULL)
        hipLaunchKernelGGL((k_nn_layer<IO_EVEN, IO_FULL>), grid, block, 0, s, L, thin, in, out, A, in_step, out_step);
    else if (inm == IO_FULL && outm == IO_EVEN)
        hipLaunchKernelGGL((k_nn_layer<IO_FULL, IO_EVEN>), grid, block, 0, s, L, thin, in, out, A, in_step, out_step);
    else
        hipLaunchKernelGGL((k_nn_layer<IO_EVEN, IO_EVEN>), grid, block, 0, s, L, thin, in, out, A, in_step, out_step);
    HISQ_HIP_CHECK(hipGetLastError());
    return HISQ_OK;
}

int nn_wgrad(const NnGeom &G, const void *thin, int cin, int cout, int inm, int gm, const void *in, const void *grad,
             int samples, size_t in_step, size_t grad_step, float *partial, double *red, size_t red_step,
             hipStream_t s) {
    const Lex L = lex_of(G);
    const int nblk = grid_blocks(gm == IO_FULL ? G.V : G.V / 2);
    const dim3 grid(nblk, samples), block(64 * NN_WAVES);
    if (inm == IO_FULL && gm == IO_FULL)
        hipLaunchKernelGGL((k_nn_wgrad<IO_FULL, IO_FULL>), grid, block, 0, s, L, thin, in, grad, partial, in_step, grad_step);
    else if (inm == IO_EVEN && gm == IO_FULL)
        hipLaunchKernelGGL((k_nn_wgrad<IO_EVEN, IO_FULL>), grid, block, 0, s, L, thin, in, grad, partial, in_step, grad_step);
    else if (inm == IO_FULL && gm == IO_EVEN)
        hipLaunchKernelGGL((k_nn_wgrad<IO_FULL, IO_EVEN>), grid, block, 0, s, L, thin, in, grad, partial, in_step, grad_step);
    else
        hipLaunchKernelGGL((k_nn_wgrad<IO_EVEN, IO_EVEN>), grid, block, 0, s, L, thin, in, grad, partial, in_step, grad_step);
    const int nent = 16 * (inm == IO_EVEN ? 16 : 80);
    float *fold = partial + (size_t)samples * grid_blocks(G.V) * 16 * 80;
    hipLaunchKernelGGL(k_nn_wgrad_fold, dim3((nent + 255) / 256, NN_FOLD, samples), dim3(256), 0, s, partial, nblk,
                       nent, fold);
    const int n = cout * 9 * cin;
    hipLaunchKernelGGL(k_nn_wgrad_reduce, dim3((n + 63) / 64, samples), dim3(64), 0, s, fold, inm, cin, cout, red,
                       red_step);
    HISQ_HIP_CHECK(hipGetLastError());
    return HISQ_OK;
}

void nn_grad_add(const double *red, int n, int samples, double *grad, const double *scal, double *loss,
                 hipStream_t s) {
    hipLaunchKernelGGL(k_nn_grad_add, dim3((n + 1 + 255) / 256), dim3(256), 0, s, red, n, samples, grad, scal, loss);
}

void nn_build_amat(const double *W, int cin, int cout, bool transposed, int inm, void *amat, hipStream_t s) {
    const int n = (int)nn_amat_elems(inm);
    hipLaunchKernelGGL(k_nn_build_amat, dim3((n + 255) / 256), dim3(256), 0, s, W, cin, cout, (int)transposed, inm,
                       (__bf16 *)amat);
}

int nn_pack_thin(const NnGeom &G, const double *U, void *dst, hipStream_t s) {
    const Lex L = lex_of(G);
    unsigned *bad = (unsigned *)((char *)dst + nn_thin_bytes(G) - 256);
    HISQ_HIP_CHECK(hipMemsetAsync(bad, 0, sizeof(unsigned), s));
    hipLaunchKernelGGL(k_pack_thin, dim3((G.V + 255) / 256, 4), dim3(256), 0, s, L, U, dst, bad);
    HISQ_HIP_CHECK(hipGetLastError());
    unsigned hb = 0;
    HISQ_HIP_CHECK(hipMemcpyAsync(&hb, bad, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    if (hb) {
        set_error("thin links: an entry is not finite or exceeds the FP16 range (|x| >= 32768)");
        return HISQ_ERR_INVALID;
    }
    return HISQ_OK;
}

void nn_loss_grad(int vh, int samples, const float *out, const float *v, float *gout, double *part, double *scal,
                  int batch, hipStream_t s) {
    const int nb = (vh + 255) / 256;
    const dim3 grid(nb, samples);
    Spinor<F32> O{const_cast<float *>(out), vh}, T{const_cast<float *>(v), vh}, Gg{gout, vh};
    hipLaunchKernelGGL(k_nn_norm2, grid, dim3(256), 0, s, T, part);
    hipLaunchKernelGGL(k_nn_scalar, dim3(samples), dim3(256), 0, s, part, nb, scal, 0, batch);
    hipLaunchKernelGGL(k_nn_loss_grad, grid, dim3(256), 0, s, O, T, scal, Gg, part);
    hipLaunchKernelGGL(k_nn_scalar, dim3(samples), dim3(256), 0, s, part, nb, scal, 1, batch);
}

void nn_adam(double *w, double *m, double *v, const double *g, int n, double lr, int step, hipStream_t s) {
    hipLaunchKernelGGL(k_nn_adam, dim3((n + 255) / 256), dim3(256), 0, s, w, m, v, g, n, lr, 0.9, 0.999, 1e-8, step);
}

}  // namespace hisq
