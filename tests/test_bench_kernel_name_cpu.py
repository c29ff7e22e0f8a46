"""The correlation kernel that bench.py names for a general rate is the one the library's
rules choose, for every N, at and just above the line in (PRN, Doppler bin) items."""
import os
import shutil
import subprocess

import pytest

import bench
from conftest import ROOT

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def test_general_rate_kernel_name(tmp_path):
    exe = str(tmp_path / "general_kernel")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-o", exe,
                    os.path.join(ROOT, "tests", "csrc", "general_kernel_driver.cpp")], check=True)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")[:-1]
    assert len(lines) == 16384
    for N, line in enumerate(lines, 1):
        _, few, many = map(int, line.split())
        for items, rows in ((256, few), (257, many)):
            assert bench.general_kernel(N, items) == ("k_gen_corr_rows" if rows else "k_gen_corr"), (N, items)
