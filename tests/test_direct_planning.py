"""The direct convolution's planning under the address and undefined-behaviour sanitizers, CPU only."""
import os
import shutil

import pytest

from test_sanitize import ROOT, _build_and_run


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_direct_planning_under_sanitizers(tmp_path):
    csrc = os.path.join(ROOT, "paper_2002_00552_amd", "csrc")
    out = _build_and_run(tmp_path, "g++",
                         [os.path.join(ROOT, "tests", "sanitize", "direct_fuzz.cpp"), os.path.join(csrc, "plan.cpp"), os.path.join(csrc, "setup.cpp")],
                         ["-std=c++17", "-Wall"], ["60"])
    assert "direct fuzz:" in out


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_direct_filter_gradient_planning_under_sanitizers(tmp_path):
    out = _build_and_run(tmp_path, "g++",
                         [os.path.join(ROOT, "tests", "sanitize", "wgrad_direct_fuzz.cpp"),
                          os.path.join(ROOT, "paper_2002_00552_amd", "csrc", "setup.cpp")],
                         ["-std=c++17", "-Wall"], ["100"])
    assert "wgrad direct fuzz:" in out
