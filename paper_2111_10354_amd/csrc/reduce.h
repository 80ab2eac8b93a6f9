// Fixed-order block reductions and the scalar steps of the CG recurrences.
#pragma once

#include "solver_internal.h"

namespace hisq {

template <class T>
__device__ __forceinline__ T wave_sum64(T v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of one double per thread over the block, in a fixed order; valid in thread 0.
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double red[16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    v = wave_sum64(v);
    if (lane == 0) red[wv] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    __syncthreads();
    return s;
}

// Sum of nb partials over the block in a fixed order; valid in thread 0.  Four
// loads of a thread are on their way at once: 10.5 -> 5.4 us for the 10368
// partials of a right-hand side on 48^3 x 12; nothing changes up to 1024.
__device__ __forceinline__ double reduce_partials(const double *part, int nb) {
    const int step = blockDim.x;
    double s = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * step < nb; i += 4 * step) {
        const double a = part[i], b = part[i + step], c = part[i + 2 * step], d = part[i + 3 * step];
        s += a;
        s += b;
        s += c;
        s += d;
    }
    for (; i < nb; i += step) s += part[i];
    return block_sum(s);
}

__device__ __forceinline__ bool finite(double v) { return v == v && fabs(v) <= 1.7e308; }

// Scalars of a running RHS from Re<p, A p>
__device__ __forceinline__ void alpha_step(CgState &S, double pap) {
    S.pap = pap;
    if (!(pap > 0.0) || !finite(pap)) {
        S.flag = CG_BREAKDOWN;
        S.xpend = 0;
    } else {
        S.alpha = S.rho / pap;
        S.xpend = 1;
    }
}

// Scalars of a running RHS from rr = |r|^2; decide: continue (beta),
// convergence check / reliable update due (host attention), or stop at the
// iteration cap.
__device__ __forceinline__ void beta_step(CgState &S, double rr) {
    S.rho_new = rr;
    S.iter += 1;
    S.since_ru += 1;
    if (!finite(rr)) {
        S.flag = CG_BREAKDOWN;
    } else if (rr <= S.stop2 || (S.ru_period > 0 && S.since_ru >= S.ru_period) || rr <= S.ru_delta2 * S.ru_rho) {
        S.flag = CG_ATTENTION;
    } else if (S.iter >= S.max_iter) {
        S.flag = CG_ATTENTION;
    } else {
        S.beta = rr / S.rho;
        S.rho = rr;
    }
}

// The sum of nb partials in every thread of the block, in reduce_partials' order.
__device__ __forceinline__ double reduce_partials_all(const double *part, int nb) {
    __shared__ double all;
    const double s = reduce_partials(part, nb);
    if (threadIdx.x == 0) all = s;
    __syncthreads();
    return all;
}

}  // namespace hisq
