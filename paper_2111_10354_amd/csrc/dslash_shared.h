// Multi-RHS Dslash whose wavefronts share a site tile's links through LDS (the
// shared shapes of hisq_internal.h; dslash_kernel.h holds the others).
//
// A workgroup of W wavefronts takes 64 output sites and W * R right-hand
// sides; each wavefront applies R of them.  The links of the tile come in
// stages of SPS slots: every wavefront loads its share of the next stage's
// units into registers while the current stage is applied, and stores them to
// the other LDS buffer at its end, so a link byte crosses the caches once for
// all right-hand sides and no thread keeps a slot's link for longer than its
// product.  The gathers of the next slots (gather_depth) are issued before the
// product of slot k.
//
// What bounds it (48^3 x 12, FP32, 16 right-hand sides: 1.15 GB, 0.157 ms at
// the 7.3 TB/s that cross the L2s; 12.2 GFLOP on the vector ALUs, 0.155 ms):
// both, and how well they overlap.  A thread with 4 RHS in its RHS tile and the
// compiler's schedule holds 185 registers (two wavefronts per SIMD) and took
// 0.436 ms in the best shape, 0.62 ms in the default one; here R = 4 takes 158
// (three wavefronts) and 0.338 ms, in FP64 0.796 ms instead of 1.78 ms.
// The tiles are swept in columns (link_tile_order): 0.45 ms in memory order.
#pragma once

#include <type_traits>
#include <utility>

#include "solver_internal.h"

namespace hisq {

// Links of a stage: SPS slots in US units (layouts of hisq_internal.h).  FP64
// groups hold one slot: two of them make a stage.
template <int LF, int CM>
struct Stage {
    static constexpr bool COMP = CM != COMP_NONE;
    static constexpr int G = LinkGroup<LF>::G;
    static constexpr int SPS = COMP ? 4 * CompGeom<LF>::MC : LF == F64 ? 2 : G;
    static constexpr int NS = 16 / SPS;
    static constexpr int US = COMP ? comp_chunk_units<LF>(CM) : SPS * 9 / G;
    static constexpr int EPU = LF == F64 ? 1 : LF == F32 ? 2 : 4;  // complex entries per unit
    // slot index (4 mu + j) of slot i of the stage, relative to the stage's first direction
    static __device__ __forceinline__ constexpr int rel_slot(int i) {
        if (!COMP) return i;
        constexpr int F = 2 * CompGeom<LF>::MC;  // fat slots first
        return i < F ? 4 * (i >> 1) + (i & 1) : 4 * ((i - F) >> 1) + 2 + ((i - F) & 1);
    }
};

// Colour vector as it lies in memory.  It is unpacked where it is used: an
// unpacking (FP16S) next to the load would wait for it there.
template <int F> struct Packed { u4v a; };
template <> struct Packed<F32> { f4v a; f2v b; };
template <> struct Packed<F64> { d2v a[3]; };

// Colour vector of site nb from a field whose base is the same for the whole
// wavefront: 32-bit byte offsets (Vh < 2^28), so one offset register serves
// every right-hand side and the bases stay in scalar registers.
template <int F>
__device__ __forceinline__ void load_packed(const char *base, int vh, unsigned nb, Packed<F> &v) {
    if constexpr (F == F64) {
        const size_t plane = (size_t)vh * 16;
#pragma unroll
        for (int c = 0; c < 3; ++c) v.a[c] = *(const d2v *)(base + c * plane + nb * 16u);
    } else if constexpr (F == F32) {
        v.a = *(const f4v *)(base + nb * 16u);
        v.b = *(const f2v *)(base + (size_t)vh * 16 + nb * 8u);
    } else {
        v.a = *(const u4v *)(base + nb * 16u);
    }
}

template <int F>
__device__ __forceinline__ void unpack(const Packed<F> &p, cx<typename RealOf<F>::T> v[3]) {
    if constexpr (F == F64) {
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = {p.a[c].x, p.a[c].y};
    } else if constexpr (F == F32) {
        v[0] = {p.a.x, p.a.y};
        v[1] = {p.a.z, p.a.w};
        v[2] = {p.b.x, p.b.y};
    } else {
        const h8v a = __builtin_bit_cast(h8v, p.a);
        const unsigned int sw = p.a.w;
        const float sc = __builtin_bit_cast(float, sw);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = {(float)a[2 * c] * sc, (float)a[2 * c + 1] * sc};
    }
}

// N complex entries from entry E0 on of the 16-byte units at `u`, ST units apart
template <int LF, int E0, int N, int ST = 64>
__device__ __forceinline__ void unit_entries(const u4v *u, cx<typename RealOf<LF>::T> *w) {
    if constexpr (LF == F64) {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const u4v raw = u[(E0 + e) * ST];
            const d2v a = __builtin_bit_cast(d2v, raw);
            w[e] = {a.x, a.y};
        }
    } else if constexpr (LF == F32) {
#pragma unroll
        for (int q = E0 / 2; q <= (E0 + N - 1) / 2; ++q) {
            const u4v raw = u[q * ST];
            const f4v a = __builtin_bit_cast(f4v, raw);
            if (2 * q >= E0 && 2 * q < E0 + N) w[2 * q - E0] = {a.x, a.y};
            if (2 * q + 1 >= E0 && 2 * q + 1 < E0 + N) w[2 * q + 1 - E0] = {a.z, a.w};
        }
    } else {
#pragma unroll
        for (int q = E0 / 4; q <= (E0 + N - 1) / 4; ++q) {
            const u4v raw = u[q * ST];
            const h8v a = __builtin_bit_cast(h8v, raw);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (4 * q + k >= E0 && 4 * q + k < E0 + N) w[4 * q + k - E0] = {(float)a[2 * k], (float)a[2 * k + 1]};
        }
    }
}

// The 3x3 matrix of slot I of a stage, its units ST apart
template <int LF, int CM, int I, int ST = 64>
__device__ __forceinline__ void stage_matrix(const u4v *u, unsigned signs, int first_mu,
                                             cx<typename RealOf<LF>::T> m[9]) {
    typedef typename RealOf<LF>::T R;
    if constexpr (CM == COMP_NONE) {
        unit_entries<LF, 9 * I, 9, ST>(u, m);
    } else {
        constexpr int F = 2 * CompGeom<LF>::MC, UF = CompGeom<LF>::UF, UL = CompGeom<LF>::UL;
        if constexpr (I < F) {
            unit_entries<LF, 9 * I, 9, ST>(u, m);
        } else {
            constexpr int L = I - F;
            unit_entries<LF, 6 * L, 6, ST>(u + UF * ST, m);
            if constexpr (CM == COMP_KAPPA) {
                cx<R> kap[1];
                unit_entries<LF, L, 1, ST>(u + (UF + UL) * ST, kap);
                rebuild_row2(m, kap[0]);
            } else {
                rebuild_row2(m, ((signs >> (2 * first_mu + L)) & 1u) ? R(-1) : R(1));
            }
        }
    }
}

template <class F, int... K>
__device__ __forceinline__ void for_slots(F &&f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K>{}), ...);
}

// An empty statement that the compiler takes to change the vector and memory:
// everything that computes the vector comes before it, every load that follows
// in the source after it.  Without it the products, which nothing needs before
// the end, are put off until all sixteen gathers of all right-hand sides are in
// registers (234 VGPRs at R = 4, or spilled).
template <class T>
__device__ __forceinline__ void settle(cx<T> v[3]) {
    asm volatile("" : "+v"(v[0].re), "+v"(v[0].im), "+v"(v[1].re), "+v"(v[1].im), "+v"(v[2].re), "+v"(v[2].im)::"memory");
}

// Slots whose gathers are in flight ahead of the product, for R right-hand
// sides of format SI per thread.  One slot against two: FP16S 28x22x18x10 with
// 5 RHS 20.4 -> 18.2 us (its records are also unpacked at the product now), FP64
// 48^3 x 12 with 8 RHS 0.448 -> 0.427 ms, FP32 there with 4 to 16 RHS the same
// within 1 %; three slots add nothing.  Not FP64 with R = 4, which holds 243
// registers already: 0.804 -> 0.921 ms.
constexpr int gather_depth(int SI, int R) { return SI == F64 && R > 3 ? 1 : 2; }

template <int LF, int SI, int SO, int R, int W, bool EPI, int CM, bool NT>
__global__ __launch_bounds__(64 * W) void dslash_shared_kernel(Geom g, const void *__restrict__ lptr, Spinor<SI> in,
                                                               Spinor<SO> out, Spinor<SI> y,
                                                               Coefs diag,
                                                               double *__restrict__ partials,
                                                               const CgState *__restrict__ skip, int parity, int nrhs,
                                                               const int *__restrict__ tiles) {
    typedef typename RealOf<LF>::T T;
    typedef Stage<LF, CM> S;
    constexpr int DEPTH = gather_depth(SI, R);
    constexpr int PU = (S::US + W - 1) / W;  // units a wavefront stages
    __shared__ u4v lds[2][S::US * 64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rb = blockIdx.y * W * R, r0 = rb + wave * R;
    if (skip) {
        bool idle = true;
        for (int r = rb; r < rb + W * R && r < nrhs; ++r)
            if (skip[r].flag == CG_RUNNING) idle = false;
        if (idle) return;  // uniform over the block
    }
    const int tile = tiles[blockIdx.x], h0 = tile * 64 + lane;
    const int h = h0 < g.vh ? h0 : g.vh - 1;  // the last tile may compute sites that it does not store
    const SiteCoord sc = decode_site(g, h, parity);
    const char *lk = (const char *)lptr + (size_t)tile * (S::NS * S::US) * 1024;
    // a wavefront, or a last tile, past the last right-hand side repeats it and
    // stores nothing
    auto rhs_of = [&](int r) { return r0 + r >= nrhs ? nrhs - 1 : r0 + r; };

    unsigned signs = 0;
    if constexpr (CM == COMP_SIGN) signs = comp_signs<LF>(lptr, g.vh, h);

    u4v pf[PU];
    auto fetch = [&](int s) {
#pragma unroll
        for (int i = 0; i < PU; ++i) {
            const int e = min(i * W + wave, S::US - 1);  // the last unit may be staged twice
            pf[i] = ldlink<NT>((const u4v *)(lk + (s * S::US + e) * 1024 + lane * 16u));
        }
    };
    auto stash = [&](int b) {
#pragma unroll
        for (int i = 0; i < PU; ++i) {
            const int e = min(i * W + wave, S::US - 1);
            lds[b][e * 64 + lane] = pf[i];
        }
    };
    // index of the neighbour of slot k = 4 mu + j
    auto neighbour = [&](int k) { return hop_index(g, sc, h, k >> 2, slot_dist(k & 3)); };
    Packed<SI> v[DEPTH + 1][R];
    auto gather = [&](int b, int k) {
        const int nb = neighbour(k);
#pragma unroll
        for (int r = 0; r < R; ++r)
            load_packed<SI>((const char *)in.rhs(rhs_of(r)).p, g.vh, (unsigned)nb, v[b][r]);
    };

    cx<T> acc[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[r][c] = {T(0), T(0)};

    // slot (4 mu + j) of the K-th of the sixteen products
    auto slot_of = [](int K) { return K / S::SPS * S::SPS + S::rel_slot(K % S::SPS); };
    // every stage and slot unrolled: no branch, so no product moves past the
    // barriers that keep one slot's gathers in flight and not all of them
    fetch(0);
    for_slots([&](auto kc) { gather(decltype(kc)::value, slot_of(decltype(kc)::value)); },
              std::make_integer_sequence<int, DEPTH>{});
    stash(0);
    __syncthreads();
    auto slot = [&](auto kc) {
        constexpr int K = decltype(kc)::value, s = K / S::SPS, I = K % S::SPS;
        if constexpr (I == 0 && s + 1 < S::NS) fetch(s + 1);
        if constexpr (K + DEPTH < 16) gather((K + DEPTH) % (DEPTH + 1), slot_of(K + DEPTH));
        __builtin_amdgcn_sched_barrier(0);
        cx<T> m[9];
        stage_matrix<LF, CM, I>(&lds[s & 1][lane], signs, s * S::SPS / 4, m);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cx<T> x[3];
            unpack<SI>(v[K % (DEPTH + 1)][r], x);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) cmac(acc[r][a], m[3 * a + b], x[b]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) settle(acc[r]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (I == S::SPS - 1 && s + 1 < S::NS) {
            stash((s + 1) & 1);
            __syncthreads();
        }
    };
    for_slots(slot, std::make_integer_sequence<int, 16>{});

#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r0 + r >= nrhs) break;
        cx<T> o[3];
        double pr = 0.0;
        if constexpr (EPI) {
            cx<T> yv[3];
            y.rhs(r0 + r).load(h, yv);
            const T d = (T)diag[r0 + r];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                o[c] = {d * yv[c].re - acc[r][c].re, d * yv[c].im - acc[r][c].im};
                pr += (double)yv[c].re * (double)o[c].re + (double)yv[c].im * (double)o[c].im;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) o[c] = acc[r][c];
        }
        typedef typename RealOf<SO>::T RO;
        cx<RO> oo[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) oo[c] = {(RO)o[c].re, (RO)o[c].im};
        if (h0 < g.vh) out.rhs(r0 + r).store_nt(h, oo);
        if constexpr (EPI) {
            if (partials) {  // a right-hand side belongs to one wavefront: its sum is the block's
                if (h0 >= g.vh) pr = 0.0;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) pr += __shfl_xor(pr, off, 64);
                if (lane == 0) partials[(size_t)(r0 + r) * gridDim.x + blockIdx.x] = pr;
            }
        }
    }
}

template <int LF, int SI, int SO, int R, int W, bool EPI>
static void launch_shared_comp(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    const dim3 grid((g.vh + 63) / 64, (a.nrhs + R * W - 1) / (R * W)), block(64 * W);
    const Spinor<SI> in = spinor_view<SI>(const_cast<void *>(a.in), g.vh);
    const Spinor<SO> out = spinor_view<SO>(a.out, g.vh);
    const Spinor<SI> y = spinor_view<SI>(const_cast<void *>(a.y ? a.y : a.in), g.vh);
    auto go = [&](auto cm) {
        constexpr int CM = decltype(cm)::value;
        if (a.cached)
            hipLaunchKernelGGL((dslash_shared_kernel<LF, SI, SO, R, W, EPI, CM, false>), grid, block, 0, s, g, a.links,
                               in, out, y, a.diag, a.partials, a.skip, a.parity, a.nrhs, a.tiles);
        else
            hipLaunchKernelGGL((dslash_shared_kernel<LF, SI, SO, R, W, EPI, CM, true>), grid, block, 0, s, g, a.links,
                               in, out, y, a.diag, a.partials, a.skip, a.parity, a.nrhs, a.tiles);
    };
    if constexpr (LF != F64) {  // FP64 links are always stored whole
        if (a.compressed == COMP_SIGN) return go(std::integral_constant<int, COMP_SIGN>{});
        if (a.compressed == COMP_KAPPA) return go(std::integral_constant<int, COMP_KAPPA>{});
    }
    go(std::integral_constant<int, COMP_NONE>{});
}

template <int LF, int SI, int SO, int R, int W>
static int launch_shared_rw(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    if (a.epilogue) launch_shared_comp<LF, SI, SO, R, W, true>(g, a, s);
    else launch_shared_comp<LF, SI, SO, R, W, false>(g, a, s);
    return 0;
}

// The (R, W) that pick_shape and the autotuner use, -1 for others.
template <int LF, int SI, int SO>
int launch_shared_fmt(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    switch (a.tile * 10 + shared_waves(a.order)) {
        case 12: return launch_shared_rw<LF, SI, SO, 1, 2>(g, a, s);
        case 13: return launch_shared_rw<LF, SI, SO, 1, 3>(g, a, s);
        case 14: return launch_shared_rw<LF, SI, SO, 1, 4>(g, a, s);
        case 23: return launch_shared_rw<LF, SI, SO, 2, 3>(g, a, s);
        case 24: return launch_shared_rw<LF, SI, SO, 2, 4>(g, a, s);
        case 33: return launch_shared_rw<LF, SI, SO, 3, 3>(g, a, s);
        case 34: return launch_shared_rw<LF, SI, SO, 3, 4>(g, a, s);
        case 44: return launch_shared_rw<LF, SI, SO, 4, 4>(g, a, s);
        default: return -1;
    }
}

}  // namespace hisq
