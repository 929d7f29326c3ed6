"""Kernel limits are found for each device of a process (csrc/per_device.hpp): the
helper under AddressSanitizer and UBSan with two devices that answer differently."""
import os

from .test_sanitizers_cpu import ROOT, _build_and_run


def test_each_device_is_asked(tmp_path):
    out = _build_and_run(tmp_path, "g++", "-std=c++20", ["tests/sanitize/per_device_check.cpp"],
                         ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_1512_04629_amd/csrc"), "-pthread"])
    assert "ok" in out
