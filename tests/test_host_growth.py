"""Growth factors at every scale factor, on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_11847_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_growth_at_every_scale_factor(tmp_path):
    exe = tmp_path / "host_growth_check"
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", f"-I{CSRC}",
           f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "host_growth_check.cpp"),
           os.path.join(CSRC, "cosmo.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)   # (an endless integration ends here)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "growth check ok" in r.stdout
