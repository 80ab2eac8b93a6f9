// Packing of the caller's canonical links into the Dslash layout.
//
// For output parity p and output site h the 16 slots k = 4 mu + j hold the
// matrix that multiplies the neighbour colour vector:
//   j = 0: F_mu(x)            (neighbour x + mu)
//   j = 1: -F_mu(x - mu)^+    (neighbour x - mu)
//   j = 2: L_mu(x)            (neighbour x + 3 mu)
//   j = 3: -L_mu(x - 3 mu)^+  (neighbour x - 3 mu)
// so the kernel is a plain 16-term gather/mat-vec sum.  Every link therefore
// appears twice in memory (once per parity it serves), which trades HBM
// capacity for fully contiguous per-site reads.
//
// One pass over the links writes every precision.  A block takes a tile of 64
// output sites, wavefront mu the four slots of direction mu.  The caller's
// layout has a link in 144 consecutive bytes and the wavefront's links 1152
// bytes apart, so a wavefront loads its 64 matrices together (nine lanes per
// link) and transposes them in LDS; every store is then 1 KiB in one piece.
// What bounds it is the traffic: each link read twice (once per parity), each
// packed byte written once, 8.1 GB on 48^3 x 12 in three precisions.  48^3 x 12
// (FP64, FP32, FP16, complex factors): 2.02 ms (4.0 TB/s, reads and writes; a
// plain copy reaches 4.7), against 11.8 ms in six launches that loaded and
// stored link by link.

#include "solver_internal.h"

namespace hisq {

typedef unsigned int u2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int64_t lex_of(const Geom &g, int x, int y, int z, int t) {
    return x + (int64_t)g.L[0] * (y + (int64_t)g.L[1] * (z + (int64_t)g.L[2] * t));
}

__device__ inline cx<double> det3(const cx<double> w[9]) {
    const cx<double> a = cmul(w[4], w[8]), b = cmul(w[5], w[7]);
    const cx<double> c2 = cmul(w[3], w[8]), d2 = cmul(w[5], w[6]);
    const cx<double> e2 = cmul(w[3], w[7]), f2 = cmul(w[4], w[6]);
    const cx<double> t0 = cmul(w[0], {a.re - b.re, a.im - b.im}), t1 = cmul(w[1], {c2.re - d2.re, c2.im - d2.im}),
                     t2 = cmul(w[2], {e2.re - f2.re, e2.im - f2.im});
    return {t0.re - t1.re + t2.re, t0.im - t1.im + t2.im};
}

// The 64 matrices of a wavefront, lane l's at field + 9 link units (link < 0:
// none), through 576 units of LDS of its own.  Every thread of the block calls it.
__device__ __forceinline__ void load_matrices(d2v *buf, const d2v *__restrict__ field, int64_t link, cx<double> w[9]) {
    const int l = threadIdx.x & 63;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int j = i * 64 + l, k = j / 9;
        const int64_t src = __shfl(link, k, 64);
        if (src >= 0) buf[j] = field[(size_t)src * 9 + (j - 9 * k)];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const d2v v = buf[9 * l + e];
        w[e] = {v.x, v.y};
    }
}

// -U^+
__device__ __forceinline__ void negate_adjoint(cx<double> w[9]) {
    cx<double> a[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) a[i] = w[i];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) w[3 * i + j] = {-a[3 * j + i].re, a[3 * j + i].im};
}

__device__ __forceinline__ unsigned half_bits(cx<double> v) {
    // double -> float -> half, round to nearest even at each step
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f2v{(float)v.re, (float)v.im}), h2v));
}

// 18 FP16 entries of two slots into the first or the second half of nine
// units (one entry is 4 bytes: the halves meet inside the fifth unit).
__device__ __forceinline__ void store_half_pair(u4v *q, bool second, const unsigned w[18]) {
    *((u2v *)(q + 4 * 64) + (second ? 1 : 0)) = second ? u2v{w[0], w[1]} : u2v{w[16], w[17]};
    if (second) {
#pragma unroll
        for (int e = 0; e < 4; ++e) q[(5 + e) * 64] = u4v{w[4 * e + 2], w[4 * e + 3], w[4 * e + 4], w[4 * e + 5]};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e * 64] = u4v{w[4 * e], w[4 * e + 1], w[4 * e + 2], w[4 * e + 3]};
    }
}

// Packed destinations, [format][output parity]; a format without memory is
// not packed.
struct PackDst {
    void *p[3][2];
};

// CM: layout of the FP32 and FP16 copies (CompMode; see CompGeom)
template <int CM>
__global__ __launch_bounds__(256) void k_pack_links(Geom g, const d2v *__restrict__ fat, const d2v *__restrict__ lng,
                                                    PackDst dst, int per, unsigned int *maxabs_bits) {
    __shared__ d2v lds[4 * 576];
    __shared__ unsigned sign[4][64];
    const int mu = threadIdx.x >> 6, l = threadIdx.x & 63;
    d2v *buf = lds + mu * 576;
    // workgroup b runs on XCD b % 8: an eighth of the tiles each, the two
    // parities of a tile (which read the same cache lines) one after the other
    const int idx = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const int tile = idx >> 1, parity = idx & 1;
    if (tile * 64 >= g.vh) return;  // uniform over the block
    const int h = tile * 64 + l;
    const bool valid = h < g.vh;
    int64_t at[2] = {-1, -1}, back3 = -1;  // links at x, x - mu and x - 3 mu
    if (valid) {
        const SiteCoord s = decode_site(g, h, parity);
        int c[4] = {s.x, s.y, s.z, s.t};
        const int64_t x = lex_of(g, c[0], c[1], c[2], c[3]);
        const int L = mu < 2 ? (mu ? g.L[1] : g.L[0]) : (mu == 2 ? g.L[2] : g.L[3]);
        const int cm = mu < 2 ? (mu ? s.y : s.x) : (mu == 2 ? s.z : s.t);
        const int64_t stride = mu == 0 ? 1 : mu == 1 ? g.L[0] : mu == 2 ? (int64_t)g.L[0] * g.L[1]
                                                                        : (int64_t)g.L[0] * g.L[1] * g.L[2];
        at[0] = x * 4 + mu;
        at[1] = (x + (wrap(cm - 1, L) - cm) * stride) * 4 + mu;
        back3 = (x + (wrap(cm - 3, L) - cm) * stride) * 4 + mu;
    }
    u4v *d64 = (u4v *)(parity ? dst.p[F64][1] : dst.p[F64][0]), *d32 = (u4v *)(parity ? dst.p[F32][1] : dst.p[F32][0]),
        *d16 = (u4v *)(parity ? dst.p[H16][1] : dst.p[H16][0]);
    constexpr int UC = CM == COMP_KAPPA ? 16 : 15;
    float m = 0.f;
    unsigned bits = 0;
#pragma unroll 1
    for (int lk = 0; lk < 2; ++lk) {  // fat, long
        cx<float> f[18];
        unsigned hw[18];
        cx<double> kap[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            cx<double> w[9];
            load_matrices(buf, lk ? lng : fat, j == 0 ? at[0] : lk ? back3 : at[1], w);
            if (j) negate_adjoint(w);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                f[9 * j + e] = {(float)w[e].re, (float)w[e].im};
                hw[9 * j + e] = half_bits(w[e]);
                if (valid) m = fmaxf(m, fmaxf(fabsf(f[9 * j + e].re), fabsf(f[9 * j + e].im)));
            }
            if (d64 && valid) {
                u4v *q = d64 + (size_t)(tile * 16 + 4 * mu + 2 * lk + j) * 9 * 64 + l;
#pragma unroll
                for (int e = 0; e < 9; ++e) q[e * 64] = __builtin_bit_cast(u4v, d2v{w[e].re, w[e].im});
            }
            if constexpr (CM != COMP_NONE) {
                if (lk) {
                    const cx<double> det = det3(w);
                    if constexpr (CM == COMP_KAPPA) {
                        double s2 = 0.0;
#pragma unroll
                        for (int e = 0; e < 9; ++e) s2 += w[e].re * w[e].re + w[e].im * w[e].im;
                        s2 /= 3.0;
                        const double inv = 1.0 / (s2 * s2);
                        kap[j] = {det.re * inv, det.im * inv};
                    } else if (valid && det.re < 0.0) {  // determinant +-1
                        bits |= 1u << (2 * mu + j);
                    }
                }
            }
        }
        if (d32 && valid) {
            if (CM == COMP_NONE || lk == 0) {
                u4v *q = d32 + (CM == COMP_NONE ? (size_t)(tile * 8 + 2 * mu + lk) * 9 : (size_t)(tile * 4 + mu) * UC) * 64 + l;
#pragma unroll
                for (int e = 0; e < 9; ++e)
                    q[e * 64] = __builtin_bit_cast(u4v, f4v{f[2 * e].re, f[2 * e].im, f[2 * e + 1].re, f[2 * e + 1].im});
            } else {
                u4v *q = d32 + ((size_t)(tile * 4 + mu) * UC + 9) * 64 + l;
#pragma unroll
                for (int e = 0; e < 6; ++e) {  // rows 0 and 1 of both slots
                    const cx<float> a = f[e < 3 ? 2 * e : 9 + 2 * (e - 3)], b = f[e < 3 ? 2 * e + 1 : 10 + 2 * (e - 3)];
                    q[e * 64] = __builtin_bit_cast(u4v, f4v{a.re, a.im, b.re, b.im});
                }
                if constexpr (CM == COMP_KAPPA)
                    q[6 * 64] = __builtin_bit_cast(u4v, f4v{(float)kap[0].re, (float)kap[0].im, (float)kap[1].re,
                                                            (float)kap[1].im});
            }
        }
        if (d16 && valid) {
            if constexpr (CM == COMP_NONE) {
                store_half_pair(d16 + (size_t)(tile * 4 + mu) * 9 * 64 + l, lk != 0, hw);
            } else {
                u4v *q = d16 + (size_t)(tile * 2 + (mu >> 1)) * UC * 64 + l;
                if (lk == 0) {
                    store_half_pair(q, mu & 1, hw);
                } else {
                    const unsigned r[12] = {hw[0], hw[1],  hw[2],  hw[3],  hw[4],  hw[5],
                                            hw[9], hw[10], hw[11], hw[12], hw[13], hw[14]};
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        q[(9 + 3 * (mu & 1) + e) * 64] = u4v{r[4 * e], r[4 * e + 1], r[4 * e + 2], r[4 * e + 3]};
                    if constexpr (CM == COMP_KAPPA)
                        *((u2v *)(q + 15 * 64) + (mu & 1)) = u2v{half_bits(kap[0]), half_bits(kap[1])};
                }
            }
        }
    }
    if constexpr (CM == COMP_SIGN) {
        // one word per site of every tile, zero for the sites past the last
        sign[mu][l] = bits;
        __syncthreads();
        if (mu == 0) {
            const unsigned word = sign[0][l] | sign[1][l] | sign[2][l] | sign[3][l];
            const size_t tiles = (size_t)(g.vh + LINK_TILE - 1) / LINK_TILE;
            if (d32) ((unsigned *)(d32 + tiles * comp_units<F32>() * 64))[h] = word;
            if (d16) ((unsigned *)(d16 + tiles * comp_units<H16>() * 64))[h] = word;
        }
    }
    if (maxabs_bits) {  // m >= 0: bit order = value order
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        if (l == 0) atomicMax(maxabs_bits, __float_as_uint(m));
    }
}

// Deviation of each long link L from a unitary matrix with determinant +-1
// (bits[0]) and from a positive multiple of a unitary matrix (bits[1]).  A
// wavefront reads 64 links in one piece; one pair of atomics per block:
// 0.28 ms on 48^3 x 12 (1.9 ms with a thread's links apart and atomics per link).
__global__ __launch_bounds__(256) void k_long_defect(int64_t nlinks, const d2v *__restrict__ lng, unsigned *bits) {
    __shared__ d2v lds[4 * 576];
    __shared__ float red[2][4];
    const int wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (site, mu)
    cx<double> m[9];
    load_matrices(lds + wave * 576, lng, i < nlinks ? i : -1, m);
    double dev1 = 0.0, dev2 = 0.0;
    if (i < nlinks) {
        double ll[9][2];
        double s2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {  // (L L^+)_ab
                double re = 0.0, im = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const cx<double> x = m[3 * a + c], y = m[3 * b + c];
                    re += x.re * y.re + x.im * y.im;
                    im += x.im * y.re - x.re * y.im;
                }
                ll[3 * a + b][0] = re;
                ll[3 * a + b][1] = im;
                if (a == b) s2 += re;
            }
        s2 /= 3.0;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const double d = (e % 4 == 0) ? 1.0 : 0.0;
            dev1 = fmax(dev1, fmax(fabs(ll[e][0] - d), fabs(ll[e][1])));
            dev2 = fmax(dev2, fmax(fabs(ll[e][0] - d * s2), fabs(ll[e][1])));
        }
        dev2 = s2 > 0.0 ? dev2 / s2 : 1e30;
        const cx<double> det = det3(m);
        dev1 = fmax(dev1, fmax(fabs(fabs(det.re) - 1.0), fabs(det.im)));
        if (!(dev1 == dev1)) dev1 = 1e30;  // NaN: not compressible
        if (!(dev2 == dev2)) dev2 = 1e30;
    }
    float d1 = (float)fmin(dev1, 1e30), d2 = (float)fmin(dev2, 1e30);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        d1 = fmaxf(d1, __shfl_xor(d1, off, 64));
        d2 = fmaxf(d2, __shfl_xor(d2, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = d1;
        red[1][wave] = d2;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const float *r = red[threadIdx.x];
        atomicMax(bits + threadIdx.x, __float_as_uint(fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]))));
    }
}

void launch_long_link_defect(const Geom &g, const double *lng, unsigned *defect_bits, hipStream_t s) {
    const int64_t n = 8 * (int64_t)g.vh;
    hipLaunchKernelGGL(k_long_defect, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, (const d2v *)lng,
                       defect_bits);
}

int launch_pack_links(const Geom &g, const double *fat, const double *lng, void *const dst[3][2], float *maxabs_dev,
                      int comp_mode, hipStream_t s) {
    PackDst d;
    for (int f = 0; f < 3; ++f)
        for (int par = 0; par < 2; ++par) d.p[f][par] = dst[f][par];
    const int per = (2 * ((g.vh + LINK_TILE - 1) / LINK_TILE) + 7) / 8;  // (tile, parity) pairs per XCD
    const dim3 grid(8 * per), block(256);
    const d2v *f = (const d2v *)fat, *l = (const d2v *)lng;
    unsigned *mb = (unsigned *)maxabs_dev;
    if (comp_mode == COMP_SIGN)
        hipLaunchKernelGGL(k_pack_links<COMP_SIGN>, grid, block, 0, s, g, f, l, d, per, mb);
    else if (comp_mode == COMP_KAPPA)
        hipLaunchKernelGGL(k_pack_links<COMP_KAPPA>, grid, block, 0, s, g, f, l, d, per, mb);
    else
        hipLaunchKernelGGL(k_pack_links<COMP_NONE>, grid, block, 0, s, g, f, l, d, per, mb);
    HISQ_HIP_CHECK(hipGetLastError());
    return HISQ_OK;
}

}  // namespace hisq
