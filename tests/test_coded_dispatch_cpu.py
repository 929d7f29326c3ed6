"""What the pair-coded form has no kernel for is an error, not an unwritten result: a
program linked to the library asks for it (no device is needed)."""
import os
import shutil
import subprocess

import pytest

from paper_1512_04629_amd import amg

from .test_sanitizers_cpu import ROOT


def test_without_an_instance_it_throws(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no compiler or no HIP headers")
    exe = str(tmp_path / "check")
    where = os.path.dirname(amg.LIB_PATH)
    b = subprocess.run(["g++", "-std=c++20", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(where, "csrc"), os.path.join(ROOT, "tests/sanitize/coded_dispatch_check.cpp"),
                        amg.LIB_PATH, "-Wl,-rpath," + where, "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib",
                        "-Wl,--allow-shlib-undefined", "-o", exe], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "dispatch: ok" in r.stdout, r.stdout + r.stderr
