"""The plan of the fused step where unscheduled pieces have chunks of their own, and the rules of its shape: tests/sanitize/plain_pieces.cpp,
under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT, SAN


@pytest.mark.timeout(600)
def test_plain_pieces(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "plain_pieces")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2502_11058_amd", "csrc")]
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN + inc + [os.path.join(ROOT, "tests", "sanitize", "plain_pieces.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=500)
    assert r.returncode == 0 and "plain pieces ok" in r.stdout, r.stdout + r.stderr
