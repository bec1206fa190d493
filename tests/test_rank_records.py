"""The rank records of the staged forest kernels (CPU only): ranks, walks and
leaf boxes against plain walks on the fp32 rows, under the sanitizers and in
a plain build, which must build the same records."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2408_05235_amd", "csrc")
SAN = ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_rank_records(tmp_path):
    out = []
    for flags in (SAN, ["-O2"]):
        exe = str(tmp_path / ("san" if flags is SAN else "plain"))
        subprocess.run(["g++", "-std=c++17", "-ffp-contract=off", "-I", CSRC, *flags,
                        os.path.join(HERE, "rank_records_check.cpp"), os.path.join(CSRC, "host_forest.cpp"), "-o", exe],
                       check=True, capture_output=True, text=True)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=600,
                           env=dict(os.environ, UBSAN_OPTIONS="halt_on_error=1"))
        assert r.returncode == 0 and "runtime error" not in r.stderr, r.stderr[-3000:]
        out.append(re.search(r"checksum=([0-9a-f]+)", r.stdout).group(1))
    assert out[0] == out[1]
