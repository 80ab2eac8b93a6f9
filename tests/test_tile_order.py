"""The tile order of the shared Dslash launches is a permutation of the lattice's
64-site tiles on any extents, and workgroups b = x (mod 8) take consecutive
tiles of the sweep (built from the library's own header, on the CPU)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = r"""
#include <cstdio>
#include <vector>
#include "hisq_internal.h"
using namespace hisq;
static Geom geom(int a, int b, int c, int d) {
    Geom g;
    int L[4] = {a, b, c, d};
    for (int i = 0; i < 4; ++i) g.L[i] = L[i];
    g.lxh = a / 2;
    g.vh = (int)((long)a * b * c * d / 2);
    g.sy = g.lxh;
    g.sz = g.sy * b;
    g.st = g.sz * c;
    return g;
}
int main() {
    long n = 0;
    for (int a : {4, 6, 10, 20, 48, 96, 130})
        for (int b : {4, 6, 14, 48})
            for (int c : {4, 10, 26})
                for (int d : {4, 6, 12}) {
                    const Geom g = geom(a, b, c, d);
                    const int nt = (g.vh + 63) / 64;
                    std::vector<int> order(nt + 8, -1), seen(nt, 0);
                    link_tile_order(g, order.data());
                    for (int i = 0; i < nt; ++i) {
                        if (order[i] < 0 || order[i] >= nt || seen[order[i]]++) {
                            std::printf("FAILED %d %d %d %d at %d\n", a, b, c, d, i);
                            return 1;
                        }
                        ++n;
                    }
                    for (int i = nt; i < nt + 8; ++i)
                        if (order[i] != -1) {
                            std::printf("FAILED past the end %d %d %d %d\n", a, b, c, d);
                            return 1;
                        }
                }
    for (int t = 0; t <= 5; ++t)
        for (int w = 0; w <= 5; ++w)
            if (shared_built(t, w) && shared_waves(shared_order(w)) != w) return 1;
    std::printf("ok %ld\n", n);
    return 0;
}
"""


def test_link_tile_order_is_a_permutation(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "order.hip", tmp_path / "order"
    src.write_text(CODE)
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2111_10354_amd", "csrc"), "-I",
                    os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout
