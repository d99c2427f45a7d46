"""The launches of the fused step over dense arenas are planned on the host: tests/sanitize/plan.cpp drives the planning code
(ddp_plan.h) through random models, schedules and layer ranges under AddressSanitizer and UndefinedBehaviorSanitizer and
checks what the kernel relies on."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT, SAN


@pytest.mark.timeout(600)
def test_pieces_of_whole_models_and_of_layer_ranges(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "plan")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2502_11058_amd", "csrc")]
    src = os.path.join(ROOT, "tests", "sanitize", "plan.cpp")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN + inc + [src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe, "700"], capture_output=True, text=True, env=env, timeout=500)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "plan sweep ok" in r.stdout, r.stdout
