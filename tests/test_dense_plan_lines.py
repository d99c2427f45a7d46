"""The plan of the fused step over dense arenas with chunks that end on cache lines: tests/sanitize/plan_lines.cpp, under
AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT, SAN


@pytest.mark.timeout(600)
def test_pieces_on_lines(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "plan_lines")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2502_11058_amd", "csrc")]
    src = os.path.join(ROOT, "tests", "sanitize", "plan_lines.cpp")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN + inc + [src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=500)
    assert r.returncode == 0 and "plan lines ok" in r.stdout, r.stdout + r.stderr
