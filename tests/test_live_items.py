"""Host check of the batch programs' maps of live items: a fill of the device
maps that fails (its copy or its kernel) leaves no set of patches marked as
held, so that the next solve fills them again instead of walking stale or
never-written indices (tests/live_items_main.cpp drives csrc/live_items.h)."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1104_1703_amd", "csrc")


def test_failed_fill_is_not_held():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "live")
        r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                            os.path.join(HERE, "live_items_main.cpp"), "-o", exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
        assert run.returncode == 0, run.stdout + run.stderr
