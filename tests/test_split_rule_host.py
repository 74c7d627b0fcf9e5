"""The attention kernels' launch-shape rule on the host (``split_rule.h``, the code the library compiles, built with g++):
over device sizes, heads, groups, batches and lengths the partials fit the workspace, dealt workgroups are resident, and
eight waves are taken only in the range where they were measured to be faster than four."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_split_rule_over_the_range_of_shapes(tmp_path):
    exe = str(tmp_path / "split_rule")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2602_20732_amd", "csrc"),
           os.path.join(ROOT, "tests", "split_rule_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
