"""The projection tries leading parts of a queue together, each try at the cost
of scans of the whole board (CPU only): the number of tries is logarithmic in
the queue's length however wrong the guess of the part that fits is."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_queue_tries(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2408_05235_amd", "csrc"),
                    os.path.join(ROOT, "tests", "sanitize", "queue_tries_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
