"""The scratch that calls on several streams and threads share (CPU only): on
a model of the runtime, for one array and for several, any two calls that get
the same array are ordered, whatever handles name their streams, no call ends
another thread's capture, and calls that no memory is left for run without."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2408_05235_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("slots", [1, 4])
def test_scratch_pool(tmp_path, slots):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", f"-DPOOL_SLOTS={slots}",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(HERE, "fake_hip"), "-I", CSRC,
                    os.path.join(HERE, "scratch_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
