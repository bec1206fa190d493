"""What the compiler reports for the projection's kernels (CPU only, gfx950
code from hipcc).  Their admission loops are chains bound by latency: a scalar
register that does not fit is written to a vector lane and read back inside the
chain."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2408_05235_amd import build


def _resources(tmp_path, name):
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc(), *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
           "-I", build.INCLUDE, "-I", build.CSRC, "-x", "hip", os.path.join(build.CSRC, name),
           "-o", str(tmp_path / "out.o")]
    text = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    kernels, cur = {}, None
    for line in text.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = kernels.setdefault(m.group(1), {})
        m = re.search(r"remark:\s+(.+?): (\d+) \[", line)
        if m and cur is not None:
            cur[re.sub(r"\s*\[.*\]$", "", m.group(1).strip())] = int(m.group(2))
    return kernels


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="no hipcc")
def test_projection_behind_a_batch_cap_keeps_its_registers(tmp_path):
    kernels = _resources(tmp_path, "project.hip")
    # project_kernel<CAP, BD_LDS, POW2, W, A>
    found = {m.groups(): r for k, r in kernels.items()
             for m in [re.search(r"project_kernelILb([01])ELb([01])ELb([01])ELi(\d)ELi(\d)E", k)] if m}
    assert len(found) == 16
    for (cap, _, _, waves, _), r in found.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0
        if cap == "1":
            assert r["SGPRs Spill"] <= (0 if waves == "1" else 8), r
            assert r["VGPRs"] <= 48, r
