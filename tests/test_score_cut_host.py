"""The selection's score keys and its search for a cut by value, on the host: ``score_cut.h`` -- the code the kernels
compile -- built with g++ under UndefinedBehaviorSanitizer and compared with sorting, over normal scores, ties, infinities
and NaNs of either sign (a NaN score may rank anywhere; a cut that loses count over it may not)."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_keys_are_monotone_and_the_search_agrees_with_sorting(tmp_path):
    exe = str(tmp_path / "score_cut")
    cmd = ["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2602_20732_amd", "csrc"), os.path.join(ROOT, "tests", "score_cut_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
