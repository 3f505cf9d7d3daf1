"""Which tasks are written as one piece: a host-only program, see tests/sanitize/pieces_driver.cpp, under the sanitizers."""

import os
import shutil

import pytest

from .test_sanitizers import ROOT, SAN, run


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pieces_of_random_plans(tmp_path):
    exe = str(tmp_path / "pieces_driver")
    csrc = os.path.join(ROOT, "paper_2404_00242_amd", "csrc")
    run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "deft_plan.cpp"),
         os.path.join(ROOT, "tests", "sanitize", "pieces_driver.cpp"), "-lpthread", "-o", exe])
    assert "pieces checked" in run([exe])
