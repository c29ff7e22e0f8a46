"""Index rules of the general-rate path on the CPU, over every N: the code replicas
of both segments read samples 0 .. N - 1 and nothing else (an odd N's second segment
is one sample shorter than its first)."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def test_code_replicas_stay_inside_their_code(tmp_path):
    exe = str(tmp_path / "general_rate")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-o", exe,
                    os.path.join(ROOT, "tests", "csrc", "general_rate_driver.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, "N, segment, position, sample: " + res.stdout
