"""What the compiler gives the averaging kernels (its own resource report): none touches scratch memory, and only those laid out for
more replicas than they have, whose conditions take scalar registers, spill any."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_11058_amd import build


@pytest.mark.timeout(600)
def test_averaging_kernels(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    r = subprocess.run([hipcc] + build.FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                                                os.path.join(build.CSRC, "ddp_kernels_mean.hip"), "-o", str(tmp_path / "mean.o")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    seen, kernel = {}, ""
    for ln in r.stderr.splitlines():
        if m := re.search(r"remark: .*Function Name: (\S+)", ln):
            kernel = m[1]
        elif m := re.search(r"remark: .* (SGPRs Spill|VGPRs Spill|ScratchSize)[^:]*: (\d+)", ln):
            seen.setdefault(kernel, {})[m[1]] = int(m[2])
    means = {k: v for k, v in seen.items() if "mean_kernel" in k}
    assert len(means) > 50 and all(len(v) == 3 for v in means.values())
    assert {k: v for k, v in seen.items() if v["ScratchSize"] or v["VGPRs Spill"]} == {}
    # (mean_kernel<NREP, EXACT, ...>; 44 is the most that the form for 17..31 replicas has ever had)
    assert {k: v for k, v in means.items() if v["SGPRs Spill"] > (0 if re.search(r"ILi\d+ELb1E", k) else 44)} == {}
