// Dslash of small lattices (the split shape of hisq_internal.h): four wavefronts
// to 64 sites, each with the four slots of one direction (FP16 compressed links:
// the fat or the long slots of a chunk of two).
//
// What bounds it: latency.  A launch of few wavefronts leaves the chip idle, and
// one thread's sixteen slots, in the registers that a full chip allows it, are
// several round trips to memory one after another.  Here a wavefront has the links
// and the neighbours of its slots on the way at once, and the four hand the sum
// from one to the next through LDS, in the order of the other kernels, so that the
// result is theirs bit for bit.  8^4, one right-hand side: FP64 7.5 -> 5.4 us,
// FP32 5.5 -> 4.7 (whole links 6.6 -> 4.7), FP16S 5.7 -> 4.6; the smallest
// kernels of a solve take 2.3.  pick_shape has the limits.
#include "dslash_shared.h"

namespace hisq {

template <int LF, int CM>
struct Segment {
    // compressed FP16: chunks of two directions, fat slots first
    static constexpr bool HALF = CM != COMP_NONE && CompGeom<LF>::MC == 2;
    static constexpr int US = HALF ? CompGeom<LF>::UF : CM != COMP_NONE ? comp_chunk_units<LF>(CM) : 36 / (LF == F64 ? 1 : LF == F32 ? 2 : 4);
    // units of segment s: first, how many
    static __device__ __forceinline__ int first(int s) {
        return HALF ? (s >> 1) * comp_chunk_units<LF>(CM) + (s & 1) * CompGeom<LF>::UF : s * US;
    }
    static __device__ __forceinline__ int units(int s) {
        return HALF && (s & 1) ? comp_chunk_units<LF>(CM) - CompGeom<LF>::UF : US;
    }
    static constexpr int TILE_UNITS = HALF ? 2 * comp_chunk_units<LF>(CM) : 4 * US;
    // direction and hop of slot i
    static __device__ __forceinline__ int mu(int s, int i) { return HALF ? (s & ~1) + (i >> 1) : s; }
    static __device__ __forceinline__ int dist(int s, int i) {
        const int d = HALF ? ((i & 1) ? -1 : 1) : ((i & 1) ? -1 : 1) * ((i & 2) ? 3 : 1);
        return HALF && (s & 1) ? 3 * d : d;
    }
    template <int I>
    static __device__ __forceinline__ void matrix(const u4v *u, unsigned signs, int s, cx<typename RealOf<LF>::T> m[9]) {
        typedef typename RealOf<LF>::T R;
        if constexpr (!HALF) {
            stage_matrix<LF, CM, I, 1>(u, signs, s, m);
        } else if (s & 1) {
            unit_entries<LF, 6 * I, 6, 1>(u, m);
            if constexpr (CM == COMP_KAPPA) {
                cx<R> kap[1];
                unit_entries<LF, I, 1, 1>(u + CompGeom<LF>::UL, kap);
                rebuild_row2(m, kap[0]);
            } else {
                rebuild_row2(m, ((signs >> (2 * (s & ~1) + I)) & 1u) ? R(-1) : R(1));
            }
        } else {
            unit_entries<LF, 9 * I, 9, 1>(u, m);
        }
    }
};

template <int LF, int SI, int SO, bool EPI, int CM>
__global__ __launch_bounds__(256) void dslash_split_kernel(Geom g, const void *__restrict__ lptr, Spinor<SI> in,
                                                           Spinor<SO> out, Spinor<SI> y, Coefs diag,
                                                           double *__restrict__ partials,
                                                           const CgState *__restrict__ skip, int parity) {
    typedef typename RealOf<LF>::T T;
    typedef Segment<LF, CM> S;
    __shared__ cx<T> hand[3][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rhs = blockIdx.y;
    const int tile = blockIdx.x, h0 = tile * 64 + lane;
    const int h = h0 < g.vh ? h0 : g.vh - 1;  // the last tile may compute sites that it does not store
    const int flag = skip ? skip[rhs].flag : CG_RUNNING;

    const char *lk = (const char *)lptr + ((size_t)tile * S::TILE_UNITS + S::first(wave)) * 1024 + lane * 16;
    const int nu = S::units(wave);
    u4v u[S::US];
#pragma unroll
    for (int e = 0; e < S::US; ++e) u[e] = *(const u4v *)(lk + (S::HALF ? min(e, nu - 1) : e) * 1024);
    unsigned signs = 0;
    if constexpr (CM == COMP_SIGN) signs = comp_signs<LF>(lptr, g.vh, h);
    const SiteCoord sc = decode_site(g, h, parity);
    const char *src = (const char *)in.rhs(rhs).p;
    Packed<SI> v[4], yp;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        load_packed<SI>(src, g.vh, (unsigned)hop_index(g, sc, h, S::mu(wave, i), S::dist(wave, i)), v[i]);
    if constexpr (EPI) load_packed<SI>((const char *)y.rhs(rhs).p, g.vh, (unsigned)h, yp);
    if (flag != CG_RUNNING) return;  // uniform over the block

    cx<T> m[4][9], x[4][3];
    for_slots(
        [&](auto ic) {
            constexpr int I = decltype(ic)::value;
            S::template matrix<I>(u, signs, wave, m[I]);
            unpack<SI>(v[I], x[I]);
        },
        std::make_integer_sequence<int, 4>{});
    // ready before the turn begins
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int a = 0; a < 3; ++a) settle(m[i] + 3 * a);
        settle(x[i]);
    }

    cx<T> acc[3] = {{T(0), T(0)}, {T(0), T(0)}, {T(0), T(0)}};
#pragma unroll 1
    for (int turn = 0; turn < 4; ++turn) {
        if (wave == turn) {
            if (turn > 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[c] = hand[c][lane];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) cmac(acc[a], m[i][3 * a + b], x[i][b]);
            if (turn < 3) {
#pragma unroll
                for (int c = 0; c < 3; ++c) hand[c][lane] = acc[c];
            }
        }
        __syncthreads();
    }
    if (wave != 3) return;

    cx<T> o[3];
    double pr = 0.0;
    if constexpr (EPI) {
        cx<T> yv[3];
        unpack<SI>(yp, yv);
        const T d = (T)diag[rhs];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            o[c] = {d * yv[c].re - acc[c].re, d * yv[c].im - acc[c].im};
            pr += (double)yv[c].re * (double)o[c].re + (double)yv[c].im * (double)o[c].im;
        }
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = acc[c];
    }
    typedef typename RealOf<SO>::T RO;
    cx<RO> oo[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) oo[c] = {(RO)o[c].re, (RO)o[c].im};
    if (h0 < g.vh) out.rhs(rhs).store(h, oo);
    if constexpr (EPI) {
        if (partials) {
            if (h0 >= g.vh) pr = 0.0;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) pr += __shfl_xor(pr, off, 64);
            if (lane == 0) partials[(size_t)rhs * gridDim.x + tile] = pr;
        }
    }
}

template <int LF, int SI, int SO, bool EPI>
static void launch_comp(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    const dim3 grid((g.vh + 63) / 64, a.nrhs), block(256);
    const Spinor<SI> in = spinor_view<SI>(const_cast<void *>(a.in), g.vh);
    const Spinor<SO> out = spinor_view<SO>(a.out, g.vh);
    const Spinor<SI> y = spinor_view<SI>(const_cast<void *>(a.y ? a.y : a.in), g.vh);
    auto go = [&](auto cm) {
        hipLaunchKernelGGL((dslash_split_kernel<LF, SI, SO, EPI, decltype(cm)::value>), grid, block, 0, s, g, a.links,
                           in, out, y, a.diag, a.partials, a.skip, a.parity);
    };
    if constexpr (LF != F64) {  // FP64 links are always stored whole
        if (a.compressed == COMP_SIGN) return go(std::integral_constant<int, COMP_SIGN>{});
        if (a.compressed == COMP_KAPPA) return go(std::integral_constant<int, COMP_KAPPA>{});
    }
    go(std::integral_constant<int, COMP_NONE>{});
}

template <int LF, int SI, int SO>
static int launch_fmt(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    if (a.epilogue) launch_comp<LF, SI, SO, true>(g, a, s);
    else launch_comp<LF, SI, SO, false>(g, a, s);
    return 0;
}

int launch_dslash_split(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    if (a.fmt_links == F64 && a.fmt_in == F64 && a.fmt_out == F64) return launch_fmt<F64, F64, F64>(g, a, s);
    if (a.fmt_links == F32 && a.fmt_in == F32 && a.fmt_out == F32) return launch_fmt<F32, F32, F32>(g, a, s);
    if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == H16) return launch_fmt<H16, H16, H16>(g, a, s);
    if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == F32) return launch_fmt<H16, H16, F32>(g, a, s);
    if (a.fmt_links == H16 && a.fmt_in == F32 && a.fmt_out == F32) return launch_fmt<H16, F32, F32>(g, a, s);
    return -1;
}

}  // namespace hisq
