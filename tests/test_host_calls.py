"""Host logic of libqpat (state, size limits, failed allocations) on the CPU: tests/host_calls.cpp runs the library's
own host code over a HIP runtime of its own, which can fail an allocation and which records launches."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1512_02796_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(PKG, "libqpat.so")) or not shutil.which(HIPCC),
                                reason="libqpat.so not built, or no hipcc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_calls")
    r = subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-rdynamic",
                        os.path.join(ROOT, "tests", "host_calls.cpp"), "-o", exe, "-L" + PKG, "-l:libqpat.so",
                        "-Wl,-rpath," + PKG], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("case", ["guess_sides", "guess_alloc_failures", "voxel_limit_per_call",
                                  "voxel_form_after_format_0", "failed_forward_state", "failed_prior_state",
                                  "hierarchy_alloc_failures", "solve_alloc_failures", "product_alloc_failures",
                                  "failed_sources_state", "idle_solves", "resident_blocks"])
def test_host_call(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
