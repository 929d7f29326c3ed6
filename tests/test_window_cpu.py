"""The adaptive window's test as a comparison with one number (csrc/window.hpp)."""
import os

from .test_sanitizers_cpu import ROOT, _build_and_run


def test_limit_decides_as_the_factor(tmp_path):
    out = _build_and_run(tmp_path, "g++", "-std=c++17", ["tests/sanitize/window_check.cpp"],
                         ["-I" + os.path.join(ROOT, "paper_1512_04629_amd/csrc")])
    assert "window_limit: ok" in out
