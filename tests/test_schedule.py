"""Launch schedules (which chunks a whole call works on as one, how rows are cut into tasks, stage 2's records) against the
plans they are made from: a host-only program, see tests/sanitize/schedule_driver.cpp, under the sanitizers."""

import os
import shutil

import pytest

from .test_sanitizers import ROOT, SAN, run
from .test_short_chunks import ONE_ROUND, ROUNDS


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_schedules_of_random_plans(tmp_path):
    exe = str(tmp_path / "schedule_driver")
    csrc = os.path.join(ROOT, "paper_2404_00242_amd", "csrc")
    run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "deft_plan.cpp"),
         os.path.join(ROOT, "tests", "sanitize", "schedule_driver.cpp"), "-lpthread", "-o", exe])
    assert "schedules checked" in run([exe])


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_trees_of_one_round_and_of_several(tmp_path):
    # what test_short_chunks.py says of its trees: whole calls of at most or more than 512 workgroups (two to a compute unit), with
    # resident tasks of several pieces and more than three row tiles among them
    exe = str(tmp_path / "tasks_driver")
    csrc = os.path.join(ROOT, "paper_2404_00242_amd", "csrc")
    run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "deft_plan.cpp"),
         os.path.join(ROOT, "tests", "sanitize", "tasks_driver.cpp"), "-lpthread", "-o", exe])
    for d, leaves, Hq, Hkv in ONE_ROUND + ROUNDS:
        groups, wide = map(int, run([exe, *map(str, (2977, leaves, 150, Hq, Hkv, 128, 256 if d == 128 else 512, 3))]).split())
        if (d, leaves, Hq, Hkv) in ROUNDS:
            assert groups > 512 and wide > 0
        else:
            assert groups <= 512 and (wide > 0 or leaves == 20)
