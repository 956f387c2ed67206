"""What the library's calls do on the host (memory taken, kernels launched, their
order), on a stand-in HIP runtime that an executable linked to libqaoa.so defines:
tests/host/calls_check.cpp.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
ROCM_INCLUDE = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    from paper_2407_13012_amd import load_library, library_path
    load_library()
    lib = library_path()
    exe = str(tmp_path_factory.mktemp("host_calls") / "calls_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                    "-I", os.path.join(ROOT, "include"), os.path.join(HOST, "calls_check.cpp"), lib,
                    f"-Wl,-rpath,{os.path.dirname(lib)}", "-Wl,--allow-shlib-undefined", "-o", exe],
                   check=True, timeout=300)
    return exe


@pytest.mark.parametrize("name", ["pinned_results", "pinning_refused", "host_exports", "device_exports", "memory_checks",
                                  "failed_allocations", "sample_waits",
                                  "batch_without_class_scratch", "batch_phase_bound",
                                  "batch_far_sizes", "batch_streams"])
def test_host_calls(checks, name):
    out = subprocess.run([checks, name], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and f"{name} ok" in out.stdout, out.stdout + out.stderr
