"""Host check of the choice between the weight gradient's two kernels
(csrc/nn_plan.h): against measured times of both, and at the limits of the
march's grid and offsets (tests/conv_plan_main.cpp)."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1104_1703_amd", "csrc")


def test_weight_gradient_choice():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "plan")
        r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                            os.path.join(HERE, "conv_plan_main.cpp"), "-o", exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
        assert run.returncode == 0, run.stdout + run.stderr
