"""Rules of ``split_rule.h`` on the host: how many splits a page list gets, against the measured ranges, and which launches of the
fused step take its lean kernel."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_driver(tmp_path, name):
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2602_20732_amd", "csrc"), os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr


def test_lists_are_split_as_their_tiles_can_use(tmp_path):
    run_driver(tmp_path, "list_splits_driver")


def test_the_lean_step_is_for_rows_of_which_three_fit(tmp_path):
    run_driver(tmp_path, "lean_step_driver")
