"""The library's host code on the CPU, over HIP runtime calls that are noted instead of made (tests/host_model/fake_hip.hpp):
what is enqueued, where, and how much of it."""
import os
import shutil
import subprocess

import pytest

import paper_2502_15294_amd as ra

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2502_15294_amd")


def _run(tmp_path, name):
    gxx, rocm = shutil.which("g++"), os.environ.get("ROCM_PATH", "/opt/rocm")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    ra.lib()
    exe = str(tmp_path / name)
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-rdynamic", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(rocm, "include"),
                        os.path.join(ROOT, "tests", "host_model", name + ".cpp"), "-o", exe, "-L", PACKAGE, "-lround_attention",
                        "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + PACKAGE, "-Wl,-rpath-link," + os.path.join(rocm, "lib")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("name", ["store_streams", "store_routes", "store_reach", "store_grid", "prefill_workspace"])
def test_host_code(tmp_path, name):
    _run(tmp_path, name)
