"""Host check of the rule that takes the deepest small level as a matrix or
relaxes it (csrc/small_rule.h), against measured times of both forms
(tests/small_rule_main.cpp)."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1104_1703_amd", "csrc")


def test_deepest_level_choice():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "rule")
        r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                            os.path.join(HERE, "small_rule_main.cpp"), "-o", exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
        assert run.returncode == 0, run.stdout + run.stderr
