"""Host code of the library against a stand-in for the HIP runtime
(host_runtime.h), so that what it does about devices, failed allocations and
kept blocks is checked without a GPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_2111_10354_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(LIBDIR, "libhisq.so")):
        pytest.fail("libhisq.so is not built (run __graft_entry__.build())")
    exe = tmp_path_factory.mktemp("host_runtime") / "check"
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(LIBDIR, "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host_runtime_check.cpp"), "-L", LIBDIR, "-lhisq",
                    f"-Wl,-rpath,{LIBDIR}", "-rdynamic", "-o", str(exe)], check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("case", ["destroy_other_device", "failed_allocation", "training_without_memory",
                                  "kept_blocks", "create_without_host_memory", "tuner_times_the_default",
                                  "two_rhs_shapes", "network_blocks", "destroy_while_refused"])
def test_host_code(program, case):
    r = subprocess.run([str(program), case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
