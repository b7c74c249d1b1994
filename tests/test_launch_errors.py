"""A launch that fails is reported by the call that made it (CPU only: the program
in launch_errors.cpp stands in for the HIP runtime)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2408_02398_amd", "libttm.so")
TTM_EDEVICE = -3


@pytest.mark.skipif(not os.path.exists(LIB), reason="libttm.so not built")
@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_failed_launches_are_reported_by_their_call(tmp_path):
    exe = str(tmp_path / "launch_errors")
    subprocess.run(["g++", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "launch_errors.cpp"), LIB, "-o", exe,
                    "-Wl,-rpath," + os.path.dirname(LIB), "-Wl,-rpath-link,/opt/rocm/lib"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = {a: (int(b), int(c)) for a, b, c in (line.split() for line in r.stdout.splitlines())}
    assert len(got) == 6
    for name, (status, left) in got.items():
        assert left == 0, name      # nothing is left for the next caller to find
        assert status == (TTM_EDEVICE if name.endswith("/fail") else 0), name
