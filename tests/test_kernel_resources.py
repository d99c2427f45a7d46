"""What the compiler gives the averaging kernels (its own resource report): none touches scratch memory, and only those laid out for
more replicas than they have, whose conditions take scalar registers, spill any.  And the table-driven fused kernels of up to 16 and of 32
replicas: their single elements' code does not keep the peers' pointers in scalar registers over the vector loop."""
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


# the fused kernel's source with the instances of a few replica counts in place of all
FUSED = """
#define DDP_FUSED_ADAM 0
#include "ddp_fused.h"
namespace ddp { namespace {
template <bool A, class K> int few(const FusedLaunch &f, const K &k) {
    return k.template go<A, false, false, 8, true, true, false, false, false>(0) + k.template go<A, false, false, 8, false, true, true, false, false>(0) +
           k.template go<A, false, false, 16, true, true, false, false, false>(0) + k.template go<A, false, false, 16, true, true, true, false, true>(0) +
           k.template go<A, false, false, 16, false, true, true, false, false>(0) + k.template go<A, false, false, 32, true, true, false, false, false>(0) +
           k.template go<A, false, false, 32, true, true, true, false, true>(0) + k.template go<A, false, false, 16, true, true, false, true, false>(0);
} } }
#define dispatch_fused few
#include "ddp_kernels_fused.hip"
"""


@pytest.mark.timeout(600)
def test_fused_kernels(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    (tmp_path / "few.hip").write_text(FUSED)
    r = subprocess.run([hipcc] + build.FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c", str(tmp_path / "few.hip"),
                                                "-o", str(tmp_path / "few.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    seen, kernel = {}, ""
    for ln in r.stderr.splitlines():
        if m := re.search(r"remark: .*Function Name: (\S+)", ln):
            kernel = m[1]
        elif m := re.search(r"remark: .* (SGPRs Spill|VGPRs Spill|ScratchSize|Occupancy)[^:]*: (\d+)", ln):
            seen.setdefault(kernel, {})[m[1]] = int(m[2])
    assert len(seen) == 8 and all("fused_kernel" in k and len(v) == 4 for k, v in seen.items())
    # SGD on 16 fp32 replicas: four workgroups per CU, the average first and the update first, for one register of the latter
    sixteen = [v for k, v in seen.items() if re.search(r"Li16ELb1ELb1ELb0ELb[01]ELb0E", k)]
    assert len(sixteen) == 2 and all(v["Occupancy"] == 4 for v in sixteen)
    assert {k: v for k, v in seen.items() if v["VGPRs Spill"] > (v in sixteen) or v["ScratchSize"] > 8 * v["VGPRs Spill"]} == {}
    # two scalar registers a peer: 28 to 99 with the pointers kept, at most 26 with eight of them read at a time
    assert {k: v["SGPRs Spill"] for k, v in seen.items() if v["SGPRs Spill"] > 27} == {}
