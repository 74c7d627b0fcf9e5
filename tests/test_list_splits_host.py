"""How many splits a page list gets (``split_rule.h``), on the host, against the measured ranges."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lists_are_split_as_their_tiles_can_use(tmp_path):
    exe = str(tmp_path / "list_splits")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2602_20732_amd", "csrc"), os.path.join(ROOT, "tests", "list_splits_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
