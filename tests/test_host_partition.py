"""The geometry of the partition of scattered particles, on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_partition_geometry(tmp_path):
    exe = tmp_path / "host_partition_check"
    cmd = ["/opt/rocm/bin/hipcc", "-x", "hip", "-std=c++17", "-O1", "--offload-arch=gfx950",
           f"-I{os.path.join(ROOT, 'paper_2010_11847_amd', 'csrc')}", f"-I{os.path.join(ROOT, 'include')}",
           os.path.join(ROOT, "tests", "host_partition_check.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert "partition geometry ok" in r.stdout
