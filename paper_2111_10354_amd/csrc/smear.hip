// HISQ link smearing on the GPU in FP64 (the HISQ action of Follana et al.,
// Phys. Rev. D 75 (2007) 054502, which the paper's code simulates, Sec. 1):
//
//   level 1   V = fat7[U]:  c1 U + c3 sum S_nu[U] + c5 sum S_rho[S_nu[U]]
//                           + c7 sum S_sig[S_rho[S_nu[U]]],  (1/8, 1/16, 1/64, 1/384)
//   U(3)      W = V (V^+ V)^(-1/2)
//   level 2   X = fat7[W] with one-link 1 and the Lepage term -1/8 sum S2_nu[W]
//   Naik      L_mu(x) = -1/24 W_mu(x) W_mu(x+mu) W_mu(x+2mu)
//
// S_nu[A]_mu(x) = T_nu(x) A_mu(x+nu) T_nu(x+mu)^+ + T_nu(x-nu)^+ A_mu(x-nu) T_nu(x-nu+mu)
// is the staple of the links A of direction mu transported along +-nu by the
// links T of the level (U, then W); S2 uses two-link transports and shifts.
// Every sum runs over distinct directions different from mu, every ordering.
//
// The staple is linear in A, so a level is three passes per direction mu, 12
// staples instead of the 15 of the nested sums (the sums of an inner level
// share the outer staple):
//   T_nu  = S_nu[U_mu]                                          (3 staples)
//   B_sig = c3 U_mu + c5 (T_nu + T_rho) + c7 (S_rho[T_nu] + S_nu[T_rho])   (6)
//   V_mu  = c1 U_mu + sum_sig S_sig[B_sig]  (+ Lepage)           (3)
// with {nu, rho, sig} the three directions other than mu.  The first two
// passes run one thread per (site, result); the third one thread per site,
// and ends in the U(3) projection (level 1) or in the phase folding and the
// canonical store (level 2).
//
// What bounds it: 50 000 FP64 fused multiply-adds per site (1.8 ms on
// 48^3 x 12 at the card's 73 TFLOP/s) against 29 KB of fields per site that
// the passes exchange through memory (38 GB, 5 ms at the 7.3 TB/s that cross
// the L2s at most), so what misses the L2s.  Hence:
//   * fields are stored entry by entry in tiles of 64 sites (below): every
//     load of a wavefront is 1 KiB in one piece, where the caller's layout
//     (576 bytes from site to site) touches 64 cache lines per load;
//   * sites are swept in columns along t, an eighth of the sweep per XCD
//     (Sweep): 48^3 x 12 in 13.2 ms against 14.7 ms with whole (z, t) planes (in
//     the same run);
//   * a staple issues the loads of five matrices before its first product and
//     the kernels take the registers for that (one or two wavefronts per
//     SIMD).  Scheduled by the compiler at three or four wavefronts it was
//     15.4 ms: each of ~20 waits was a round trip, and the sites in flight
//     did not fit the L2 (T pass: 2.85 GB from beyond the L2, now 1.2 GB).
// 48^3 x 12: 51 ms in 150 canonical-layout launches before, 12.7 ms now
// (T 0.33, B 0.67, V 0.39 and 0.68 with Lepage, each 4 times per level);
// 96^3 x 24: 840 ms before, 204 ms now.
//
// Scratch: the two outputs hold intermediate fields until their own pass
// writes them, and one workspace of six one-direction fields comes on top:
//   level 1: fat = tiled U, lng and ws[4..5] = T and B, ws[0..3] = W
//   level 2: ws[0..3] = W, lng and ws[4..5] = T and B, fat = X (result)
//   Naik:    lng from ws[0..3].

#include <algorithm>
#include <cmath>

#include "solver_internal.h"

namespace hisq {

namespace {

struct M3 {
    cx<double> e[9];
};

__device__ __forceinline__ M3 mul(const M3 &a, const M3 &b) {  // a b
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(s, a.e[3 * i + k], b.e[3 * k + j]);
            r.e[3 * i + j] = s;
        }
    return r;
}

__device__ __forceinline__ cx<double> conjc(cx<double> a) { return {a.re, -a.im}; }

__device__ __forceinline__ M3 mul_an(const M3 &a, const M3 &b) {  // a^+ b
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(s, conjc(a.e[3 * k + i]), b.e[3 * k + j]);
            r.e[3 * i + j] = s;
        }
    return r;
}

__device__ __forceinline__ M3 mul_na(const M3 &a, const M3 &b) {  // a b^+
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(s, a.e[3 * i + k], conjc(b.e[3 * j + k]));
            r.e[3 * i + j] = s;
        }
    return r;
}

__device__ __forceinline__ M3 zero3() {
    M3 r;
#pragma unroll
    for (int i = 0; i < 9; ++i) r.e[i] = {0.0, 0.0};
    return r;
}

// r += a b and r += a b^+
__device__ __forceinline__ void mac3(M3 &r, const M3 &a, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(r.e[3 * i + j], a.e[3 * i + k], b.e[3 * k + j]);
}

__device__ __forceinline__ void mac3_na(M3 &r, const M3 &a, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(r.e[3 * i + j], a.e[3 * i + k], conjc(b.e[3 * j + k]));
}

__device__ __forceinline__ void axpy3(M3 &r, double c, const M3 &a) {
#pragma unroll
    for (int i = 0; i < 9; ++i) r.e[i] = {fma(c, a.e[i].re, r.e[i].re), fma(c, a.e[i].im, r.e[i].im)};
}

struct Lat {
    int L[4];
    int st[4];  // index strides
    int V;
};

// One-direction field of 9 V complex entries in tiles of 64 sites: entry e of
// site s at unit (s / 64) * 576 + e * w + s % 64, w = the tile's sites (64, or
// V % 64 in a last partial tile), so a field takes exactly 144 V bytes.
__device__ __forceinline__ M3 load3(const d2v *f, const Lat &lat, int s) {
    const int tile = s >> 6, rest = lat.V - (tile << 6), w = rest < 64 ? rest : 64;
    const d2v *q = f + (size_t)tile * 576 + (s & 63);
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const d2v v = q[e * w];
        m.e[e] = {v.x, v.y};
    }
    return m;
}

__device__ __forceinline__ void store3(d2v *f, const Lat &lat, int s, const M3 &m) {
    const int tile = s >> 6, rest = lat.V - (tile << 6), w = rest < 64 ? rest : 64;
    d2v *q = f + (size_t)tile * 576 + (s & 63);
#pragma unroll
    for (int e = 0; e < 9; ++e) q[e * w] = d2v{m.e[e].re, m.e[e].im};
}

// Site of a thread.  The sites are swept in columns of `by` y-rows by `bz`
// z-planes along t (the last column of a row may be narrower).  Workgroup b
// runs on XCD b % 8 and gets a contiguous eighth of the sweep, with the `nvar`
// variants of a site block (the results of one pass) back to back on the same
// XCD, where they share their inputs.
struct Sweep {
    int nb, per, nvar;  // site blocks, site blocks per XCD, variants
    int by, bz;
};

struct Site {
    int s;  // lexicographic index
    int c[4];
    int var;
    bool valid;
    __device__ __forceinline__ int coord(int d) const { return d < 2 ? (d ? c[1] : c[0]) : (d == 2 ? c[2] : c[3]); }
    // index offset of the site k steps along d (|k| < L[d])
    __device__ __forceinline__ int step(const Lat &lat, int d, int k) const {
        const int q = coord(d) + k, L = lat.L[d];
        return (q < 0 ? k + L : q >= L ? k - L : k) * lat.st[d];
    }
};

// `local`: the thread's site in its block of `bsites`.
__device__ __forceinline__ Site sweep_site(const Lat &lat, const Sweep &sw, int local, int bsites) {
    Site x;
    const int q = blockIdx.x >> 3;
    x.var = q % sw.nvar;
    const int blk = (blockIdx.x & 7) * sw.per + q / sw.nvar;
    const unsigned i = (unsigned)blk * bsites + local;
    x.valid = q / sw.nvar < sw.per && blk < sw.nb && i < (unsigned)lat.V;
    const unsigned slab = (unsigned)lat.st[2] * lat.L[3] * sw.bz;
    unsigned r = x.valid ? i : 0u;
    const int zb = (int)(r / slab), z0 = zb * sw.bz, wz = min(sw.bz, lat.L[2] - z0);
    r -= zb * slab;
    const unsigned col = (unsigned)lat.L[0] * sw.by * wz * lat.L[3];
    const int yb = (int)(r / col), y0 = yb * sw.by, wy = min(sw.by, lat.L[1] - y0);
    r -= yb * col;
    const unsigned row = (unsigned)lat.L[0] * wy, slice = row * wz;
    x.c[3] = (int)(r / slice);
    r -= x.c[3] * slice;
    const unsigned zz = r / row;
    r -= zz * row;
    const unsigned yy = r / (unsigned)lat.L[0];
    x.c[0] = (int)(r - yy * lat.L[0]);
    x.c[1] = y0 + (int)yy;
    x.c[2] = z0 + (int)zz;
    x.s = x.c[0] + x.c[1] * lat.st[1] + x.c[2] * lat.st[2] + x.c[3] * lat.st[3];
    return x;
}

// The three directions other than mu.
__device__ __forceinline__ int other(int mu, int k) { return k < mu ? k : k + 1; }

// Nothing moves across: the loads above it are all issued before the
// arithmetic below.  Left to itself the compiler, short of registers, loads a
// matrix, waits and multiplies, one round trip of memory after another.
#define LOADS_FIRST() __builtin_amdgcn_sched_barrier(0)

// acc += S_nu[A]_mu at site x; T: transports of direction nu
__device__ __forceinline__ void staple(M3 &acc, const Lat &lat, const Site &x, const d2v *T, const d2v *A, int mu,
                                       int nu) {
    const int up = x.s + x.step(lat, nu, 1), dn = x.s + x.step(lat, nu, -1), sm = x.step(lat, mu, 1);
    const M3 a = load3(T, lat, x.s), b = load3(A, lat, up), c = load3(T, lat, x.s + sm);
    const M3 d = load3(T, lat, dn), e = load3(A, lat, dn);
    LOADS_FIRST();
    const M3 p = mul(a, b);
    const M3 f = load3(T, lat, dn + sm);
    LOADS_FIRST();
    mac3_na(acc, p, c);
    mac3(acc, mul_an(d, e), f);
}

// acc += the two-step staple S2_nu[A]_mu at site x
__device__ __forceinline__ void staple2(M3 &acc, const Lat &lat, const Site &x, const d2v *T, const d2v *A, int mu,
                                        int nu) {
    const int sm = x.step(lat, mu, 1), up = x.s + x.step(lat, nu, 1), up2 = x.s + x.step(lat, nu, 2);
    const int dn = x.s + x.step(lat, nu, -1), dn2 = x.s + x.step(lat, nu, -2);
    {
        const M3 a = load3(T, lat, up), b = load3(A, lat, up2), c = load3(T, lat, x.s);
        const M3 d = load3(T, lat, up + sm), e = load3(T, lat, x.s + sm);
        LOADS_FIRST();
        mac3_na(acc, mul_na(mul(c, mul(a, b)), d), e);
    }
    const M3 a = load3(T, lat, dn2), b = load3(A, lat, dn2), c = load3(T, lat, dn);
    const M3 d = load3(T, lat, dn2 + sm), e = load3(T, lat, dn + sm);
    LOADS_FIRST();
    mac3(acc, mul(mul_an(c, mul_an(a, b)), d), e);
}

// The six one-direction scratch fields of a level: T and B of the directions
// other(mu, 0..2).
struct Scratch {
    d2v *t[3], *b[3];
};

// Canonical links [V][4][3][3] to four tiled fields, through LDS: a wavefront
// reads the 18 KiB of its 32 sites in one piece.
constexpr int TILE_LD = 37;  // units per site in LDS: 36 and one against bank conflicts
__global__ __launch_bounds__(64) void k_to_tiles(Lat lat, const d2v *__restrict__ src, d2v *__restrict__ dst) {
    __shared__ d2v buf[32 * TILE_LD];
    const int s0 = blockIdx.x * 32, l = threadIdx.x, n = min(32, lat.V - s0);
    const d2v *q = src + (size_t)s0 * 36;
#pragma unroll
    for (int i = 0; i < 18; ++i) {
        const int j = i * 64 + l;
        if (j < n * 36) buf[(j / 36) * TILE_LD + j % 36] = __builtin_nontemporal_load(q + j);
    }
    __syncthreads();
    const int site = l & 31, k0 = (l >> 5) * 18;  // half a wavefront per pair of directions
    if (site >= n) return;
    const int s = s0 + site, tile = s >> 6, w = min(64, lat.V - (tile << 6));
#pragma unroll
    for (int k = 0; k < 18; ++k) {
        const int mu = (k0 + k) / 9, e = (k0 + k) % 9;
        dst[((size_t)mu * lat.V + (size_t)tile * 64) * 9 + e * w + (s & 63)] = buf[site * TILE_LD + k0 + k];
    }
}

// m into direction mu of a canonical field, through LDS (576 units per
// wavefront): each site's nine units leave as one run.  Every thread of the
// block calls it.
__device__ __forceinline__ void put_canonical(d2v *buf, d2v *out, const Site &x, int mu, const M3 &m) {
    const int l = threadIdx.x & 63;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 9; ++e) buf[9 * l + e] = d2v{m.e[e].re, m.e[e].im};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int j = i * 64 + l, k = j / 9;
        const int s = __shfl(x.valid ? x.s : -1, k, 64);
        if (s >= 0) __builtin_nontemporal_store(buf[j], out + ((size_t)s * 4 + mu) * 9 + (j - 9 * k));
    }
}

// pass 1: T_nu = S_nu[U_mu], nu = other(mu, variant)
__global__ __launch_bounds__(256) void k_fat7_t(Lat lat, Sweep sw, const d2v *__restrict__ U, Scratch f, int mu) {
    const Site x = sweep_site(lat, sw, threadIdx.x, blockDim.x);
    if (!x.valid) return;
    const size_t dir = (size_t)9 * lat.V;
    const int nu = other(mu, x.var);
    M3 acc = zero3();
    staple(acc, lat, x, U + nu * dir, U + mu * dir, mu, nu);
    store3(f.t[x.var], lat, x.s, acc);
}

// pass 2: B_sig, sig = other(mu, variant), from U_mu and the T of the other two
__global__ __launch_bounds__(256) void k_fat7_b(Lat lat, Sweep sw, const d2v *__restrict__ U, Scratch f, int mu,
                                                double c3, double c5, double c7) {
    const Site x = sweep_site(lat, sw, threadIdx.x, blockDim.x);
    if (!x.valid) return;
    const size_t dir = (size_t)9 * lat.V;
    const int k0 = x.var == 0 ? 1 : 0, k1 = x.var == 2 ? 1 : 2;
    const int nu = other(mu, k0), rho = other(mu, k1);
    M3 acc = zero3();
#pragma unroll 1
    for (int k = 0; k < 2; ++k)
        staple(acc, lat, x, U + (k ? nu : rho) * dir, f.t[k ? k1 : k0], mu, k ? nu : rho);
#pragma unroll
    for (int e = 0; e < 9; ++e) acc.e[e] = {c7 * acc.e[e].re, c7 * acc.e[e].im};
    axpy3(acc, c5, load3(f.t[k0], lat, x.s));
    axpy3(acc, c5, load3(f.t[k1], lat, x.s));
    axpy3(acc, c3, load3(U + mu * dir, lat, x.s));
    store3(f.b[x.var], lat, x.s, acc);
}

// W = V (V^+ V)^(-1/2) of one matrix.  With the
// eigenvalues l_i = s_i^2 of Q = V^+ V (all positive), Q^(-1/2) = f0 + f1 Q +
// f2 Q^2 where the f's interpolate 1/s at the three s_i; in terms of u = sum
// s_i, v = sum_{i<j} s_i s_j, w = prod s_i (so that the denominators carry
// u v - w = (s0+s1)(s0+s2)(s1+s2) > 0 and stay finite for equal eigenvalues):
//   f2 = u / d,  f1 = (2 u v - w - u^3) / d,  f0 = (v (u v - w) - w u^2) / d,
//   d = w (u v - w).
__device__ __forceinline__ M3 u3_project(const M3 &v) {
    const M3 q = mul_an(v, v);
    // eigenvalues of the Hermitian Q: trigonometric solution of the cubic
    const double m = (q.e[0].re + q.e[4].re + q.e[8].re) / 3.0;
    const double k00 = q.e[0].re - m, k11 = q.e[4].re - m, k22 = q.e[8].re - m;
    const cx<double> k01 = q.e[1], k02 = q.e[2], k12 = q.e[5];
    const double n01 = k01.re * k01.re + k01.im * k01.im, n02 = k02.re * k02.re + k02.im * k02.im,
                 n12 = k12.re * k12.re + k12.im * k12.im;
    const double p = (k00 * k00 + k11 * k11 + k22 * k22 + 2.0 * (n01 + n02 + n12)) / 6.0;
    // det K for Hermitian K: real
    const cx<double> t = cmul(cmul(k01, k12), conjc(k02));
    const double detk = k00 * k11 * k22 + 2.0 * t.re - k00 * n12 - k11 * n02 - k22 * n01;
    double l[3];
    if (p <= 1e-300) {
        l[0] = l[1] = l[2] = m;
    } else {
        const double sp = sqrt(p);
        double r = detk / (2.0 * p * sp);
        r = fmin(1.0, fmax(-1.0, r));
        const double phi = acos(r) / 3.0;
        const double tpi3 = 2.0943951023931954923;  // 2 pi / 3
        l[0] = m + 2.0 * sp * cos(phi);
        l[1] = m + 2.0 * sp * cos(phi + tpi3);
        l[2] = m + 2.0 * sp * cos(phi - tpi3);
    }
    const double s0 = sqrt(fmax(l[0], 0.0)), s1 = sqrt(fmax(l[1], 0.0)), s2 = sqrt(fmax(l[2], 0.0));
    const double u = s0 + s1 + s2, vv = s0 * s1 + s0 * s2 + s1 * s2, w = s0 * s1 * s2;
    const double uvw = u * vv - w, d = w * uvw;
    const double f2 = u / d, f1 = (2.0 * u * vv - w - u * u * u) / d, f0 = (vv * uvw - w * u * u) / d;
    const M3 q2 = mul(q, q);
    M3 r;
#pragma unroll
    for (int e = 0; e < 9; ++e)
        r.e[e] = {f1 * q.e[e].re + f2 * q2.e[e].re, f1 * q.e[e].im + f2 * q2.e[e].im};
    r.e[0].re += f0;
    r.e[4].re += f0;
    r.e[8].re += f0;
    const M3 wc = mul(v, r);
    // one Newton-Schulz step towards the polar factor, W <- W (3 - W^+ W) / 2:
    // where V is badly conditioned the closed form leaves W unitary only to
    // ~eps cond(V)^2; the step squares that defect
    const M3 ww = mul_an(wc, wc);
#pragma unroll
    for (int e = 0; e < 9; ++e) r.e[e] = {-0.5 * ww.e[e].re, -0.5 * ww.e[e].im};
    r.e[0].re += 1.5;
    r.e[4].re += 1.5;
    r.e[8].re += 1.5;
    return mul(wc, r);
}

__device__ __forceinline__ double eta_sign(const int c[4], int mu) {
    int e = 0;
    for (int d = 0; d < mu; ++d) e += c[d];
    return (e & 1) ? -1.0 : 1.0;
}

// pass 3, level 1: W_mu = projection of c1 U_mu + sum_sig S_sig[B_sig]
// level 2 (Lepage weight cl): X_mu with the phase and the boundary sign
// (t + 1 >= Lt) folded in, canonical
template <int LEVEL>
__global__ __launch_bounds__(256) void k_fat7_v(Lat lat, Sweep sw, const d2v *__restrict__ U, Scratch f, int mu,
                                                double c1, double cl, d2v *__restrict__ out, int apbc) {
    __shared__ d2v buf[LEVEL == 2 ? 4 * 576 : 1];
    const Site x = sweep_site(lat, sw, threadIdx.x, blockDim.x);
    const size_t dir = (size_t)9 * lat.V;
    M3 acc = zero3();
    if (x.valid) {
        if constexpr (LEVEL == 2) {
#pragma unroll 1
            for (int k = 0; k < 3; ++k) staple2(acc, lat, x, U + other(mu, k) * dir, U + mu * dir, mu, other(mu, k));
#pragma unroll
            for (int e = 0; e < 9; ++e) acc.e[e] = {cl * acc.e[e].re, cl * acc.e[e].im};
        }
#pragma unroll 1
        for (int k = 0; k < 3; ++k) staple(acc, lat, x, U + other(mu, k) * dir, f.b[k], mu, other(mu, k));
        axpy3(acc, c1, load3(U + mu * dir, lat, x.s));
        if constexpr (LEVEL == 1) {
            store3(out + mu * dir, lat, x.s, u3_project(acc));
        } else {
            double sg = eta_sign(x.c, mu);
            if (apbc && mu == 3 && x.c[3] + 1 >= lat.L[3]) sg = -sg;
#pragma unroll
            for (int e = 0; e < 9; ++e) acc.e[e] = {sg * acc.e[e].re, sg * acc.e[e].im};
        }
    }
    if constexpr (LEVEL == 2) put_canonical(buf + (threadIdx.x >> 6) * 576, out, x, mu, acc);
}

// L_mu(x) = cN W_mu(x) W_mu(x+mu) W_mu(x+2mu), with eta_mu(x) and the time
// boundary sign (t + 3 >= Lt) folded in.  A wavefront takes 16 sites x 4
// directions and writes their 9 KiB in one piece (144-byte runs per direction
// cost a third more write traffic).
__global__ __launch_bounds__(256) void k_naik(Lat lat, Sweep sw, const d2v *__restrict__ W, d2v *__restrict__ lng,
                                              double cn, int apbc) {
    __shared__ d2v lds[4 * 16 * TILE_LD];
    const int l = threadIdx.x & 63, mu = l >> 4;
    d2v *buf = lds + (threadIdx.x >> 6) * 16 * TILE_LD;
    const Site x = sweep_site(lat, sw, (threadIdx.x >> 6) * 16 + (l & 15), 64);
    if (x.valid) {
        const d2v *Wm = W + (size_t)mu * 9 * lat.V;
        const M3 a = load3(Wm, lat, x.s), b = load3(Wm, lat, x.s + x.step(lat, mu, 1)),
                 c = load3(Wm, lat, x.s + x.step(lat, mu, 2));
        LOADS_FIRST();
        const M3 p = mul(mul(a, b), c);
        double sg = cn * eta_sign(x.c, mu);
        if (apbc && mu == 3 && x.c[3] + 3 >= lat.L[3]) sg = -sg;
#pragma unroll
        for (int e = 0; e < 9; ++e) buf[(l & 15) * TILE_LD + 9 * mu + e] = d2v{sg * p.e[e].re, sg * p.e[e].im};
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int j = i * 64 + l, k = j / 36, u = j - 36 * k;
        const int s = __shfl(x.valid ? x.s : -1, k, 64);
        if (s >= 0) __builtin_nontemporal_store(buf[k * TILE_LD + u], lng + (size_t)s * 36 + u);
    }
}

// Sites of a column's t-slice: the XCD's 32 compute units hold about 5000
// sites (half with one wavefront per SIMD), three t-slices of a column.  On
// 48^3 x 12 (Lx = 48) columns of 2 x 2, 4 x 4, 6 x 6 and 8 x 8 rows take 14.6,
// 13.9, 13.6 and 14.0 ms.
constexpr double kSweepSlice = 1728.0;
// Blocks of 256 threads; of one wavefront where 256 would leave compute units
// without a block (2^18 sites: 1024 blocks of 256).
constexpr int kSmallSweep = 1 << 18;
struct SweepLaunch {
    Sweep sw;
    dim3 grid, block;
    SweepLaunch(const Lat &lat, int nvar, unsigned bs = 0) {
        if (!bs) bs = lat.V < kSmallSweep ? 64 : 256;
        const int nb = (int)(((unsigned)lat.V + bs - 1) / bs);
        const int side = std::max(2, (int)std::lround(std::sqrt(kSweepSlice / (double)lat.L[0])));
        sw = {nb, (nb + 7) / 8, nvar, std::min(side, lat.L[1]), std::min(side, lat.L[2])};
        grid = dim3(8u * sw.per * nvar);
        block = dim3(bs);
    }
};

}  // namespace

int smear_links(const int dims[4], const double *thin, double *fat, double *lng, unsigned flags, hipStream_t s) {
    Lat lat;
    int st = 1;
    for (int i = 0; i < 4; ++i) {
        lat.L[i] = dims[i];
        lat.st[i] = st;
        st *= dims[i];
    }
    lat.V = st;
    const int apbc = (flags & HISQ_SMEAR_ANTIPERIODIC_T) ? 1 : 0;
    const size_t dir = (size_t)lat.V * 9;  // units of a one-direction field
    DevBuf ws;
    int rc;
    if ((rc = ws.alloc(6 * dir * sizeof(d2v)))) return rc;
    d2v *W = (d2v *)ws.p, *U = (d2v *)fat, *l = (d2v *)lng;
    const Scratch f{{l, l + dir, l + 2 * dir}, {l + 3 * dir, W + 4 * dir, W + 5 * dir}};
    const double c3 = 1.0 / 16, c5 = 1.0 / 64, c7 = 1.0 / 384;
    const SweepLaunch one(lat, 1), three(lat, 3), naik(lat, 1, 64);
    hipLaunchKernelGGL(k_to_tiles, dim3((lat.V + 31) / 32), dim3(64), 0, s, lat, (const d2v *)thin, U);
    for (int level = 1; level <= 2; ++level) {
        const d2v *T = level == 1 ? U : W;  // the level's links
        for (int mu = 0; mu < 4; ++mu) {
            hipLaunchKernelGGL(k_fat7_t, three.grid, three.block, 0, s, lat, three.sw, T, f, mu);
            hipLaunchKernelGGL(k_fat7_b, three.grid, three.block, 0, s, lat, three.sw, T, f, mu, c3, c5, c7);
            if (level == 1)
                hipLaunchKernelGGL(k_fat7_v<1>, one.grid, one.block, 0, s, lat, one.sw, T, f, mu, 1.0 / 8, 0.0, W, 0);
            else
                hipLaunchKernelGGL(k_fat7_v<2>, one.grid, one.block, 0, s, lat, one.sw, T, f, mu, 1.0, -1.0 / 8,
                                   (d2v *)fat, apbc);
        }
    }
    hipLaunchKernelGGL(k_naik, naik.grid, dim3(256), 0, s, lat, naik.sw, W, l, -1.0 / 24, apbc);
    HISQ_HIP_CHECK(hipGetLastError());
    // the workspace is given back on return: wait for the kernels that use it
    HISQ_HIP_CHECK(hipStreamSynchronize(s));
    ws.recycle();
    return HISQ_OK;
}

}  // namespace hisq
