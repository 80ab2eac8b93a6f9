// Host side of the Dslash: launch shapes, their checks, and the dispatch over
// the formats (kernel: dslash_kernel.h; one source file per set of formats
// holds its instances, so that they compile side by side).

#include "solver_internal.h"

namespace hisq {

Geom make_geom(const int dims[4]) {
    Geom g;
    for (int i = 0; i < 4; ++i) g.L[i] = dims[i];
    g.lxh = dims[0] / 2;
    g.vh = (int)((int64_t)dims[0] * dims[1] * dims[2] * dims[3] / 2);
    g.sy = g.lxh;
    g.sz = g.lxh * dims[1];
    g.st = g.lxh * dims[1] * dims[2];
    return g;
}

int dslash_grid_blocks(const Geom &g, int block, int order) {
    if (shared_waves(order) || order == SPLIT_ORDER) return (g.vh + 63) / 64;
    const int sb = block / order_rsplit(order);
    const int k = (order_tiles(order) & 0xff) == 4 ? (order >> 8) & 0xff : 1;  // t-march: K sites per thread
    const int threads = k > 0 ? g.vh / k : g.vh;
    return (threads + sb - 1) / sb;
}

// LDS of the x-row staging per workgroup: TILE x 3 colours x block sites
static size_t xrow_lds_bytes(int fl, int tile, int block) {
    return (size_t)tile * 3 * block * 2 * (fl == F64 ? 8 : 4);
}
static constexpr size_t kXrowLdsMax = 64 * 1024;

bool order_supported(const Geom &g, int order, int block) {
    if (order < 0 || (order >> 26)) return false;
    if (const int w = shared_waves(order)) return block == 64 * w && shared_supported(g);
    if (order == SPLIT_ORDER) return block == 256 && shared_supported(g);
    const int rs = order_rsplit(order);
    if (rs == 8 || block / rs < 64) return false;  // whole waves of sites
    // x-row staging: one wave per site, workgroups of whole rows
    if (order == 3) return (block == 64 || block == 128 || block == 192 || block == 256) && block % g.lxh == 0;
    if (block != 64 && block != 128 && block != 256) return false;
    block /= rs;
    order = order_tiles(order);
    const int kind = order & 0xff;
    if (kind == 0) return order == 0;
    if (kind == 4) {  // t-march: K sites per thread, K dividing Lt / 2
        const int k = (order >> 8) & 0xff;
        return (order >> 16) == 0 && k >= 1 && (g.L[3] / 2) % k == 0;
    }
    if (g.vh % 64 || (g.lxh * g.L[1]) % 64) return false;
    if (kind == 1) return order == 1;
    if (kind != 2 || (order >> 24)) return false;
    // whole tiles per column row block, whole blocks, and a grid of whole
    // eighths (the XCD remap is a permutation only then)
    const int by = (order >> 8) & 0xff, bz = (order >> 16) & 0xff;
    if (by < 1 || bz < 1 || g.L[1] % by || g.L[2] % bz || (g.lxh * by) % 64) return false;
    if (block < 64 || g.vh % block) return false;
    return (g.vh / block) % 8 == 0;
}

template <int LF, int SI, int SO>
int launch_epi(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_epi<F64, F64, F64>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_epi<F32, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_epi<H16, H16, H16>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_epi<H16, H16, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_epi<H16, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

int launch_dslash(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    if (shared_waves(a.order)) return launch_dslash_shared(g, a, s);
    const bool xrow = a.order == 3;
    if (a.block != 64 && a.block != 128 && a.block != 256 && !(xrow && a.block == 192)) {
        set_error("dslash: block size must be 64, 128 or 256 (or 192 with x-row staging)");
        return HISQ_ERR_INVALID;
    }
    if (!order_supported(g, a.order, a.block)) {
        set_error("dslash: traversal order not supported for this lattice");
        return HISQ_ERR_INVALID;
    }
    if (xrow && (a.tile > 8 || xrow_lds_bytes(a.fmt_links, a.tile, a.block) > kXrowLdsMax)) {
        set_error("dslash: x-row staging takes RHS tiles of at most 8 and 64 KiB of LDS");
        return HISQ_ERR_INVALID;
    }
    if ((order_tiles(a.order) & 0xff) == 4 && a.tile > 4) {
        set_error("dslash: the t-march takes RHS tiles of at most 4");
        return HISQ_ERR_INVALID;
    }
    int rc = -1;
    if (a.order == SPLIT_ORDER)
        rc = a.tile == 1 ? launch_dslash_split(g, a, s) : -1;
    else if (a.fmt_links == F64 && a.fmt_in == F64 && a.fmt_out == F64)
        rc = launch_epi<F64, F64, F64>(g, a, s);
    else if (a.fmt_links == F32 && a.fmt_in == F32 && a.fmt_out == F32)
        rc = launch_epi<F32, F32, F32>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == H16)
        rc = launch_epi<H16, H16, H16>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == F32)
        rc = launch_epi<H16, H16, F32>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == F32 && a.fmt_out == F32)
        rc = launch_epi<H16, F32, F32>(g, a, s);
    if (rc != 0) {
        set_error("dslash: unsupported precision / tile combination");
        return HISQ_ERR_UNSUPPORTED;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error(std::string("dslash launch: ") + hipGetErrorString(e));
        return HISQ_ERR_HIP;
    }
    return HISQ_OK;
}

}  // namespace hisq
