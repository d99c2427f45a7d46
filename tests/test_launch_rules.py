"""The rules that choose a launch's form: tests/sanitize/rules.cpp."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT, SAN


def test_both_sides_of_the_rules(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "rules")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2502_11058_amd", "csrc")]
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN + inc + [os.path.join(ROOT, "tests", "sanitize", "rules.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert r.returncode == 0 and "rules ok" in r.stdout, r.stdout + r.stderr
