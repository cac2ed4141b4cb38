"""Launch shapes set or tuned for a relay graph's variable launches are those
its relay iterations run with (a native program on the in-tree liblbp.so reads
them back)."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2202_04110_amd")


def test_relay_launches_take_the_set_shapes(tmp_path):
    exe = str(tmp_path / "relay_shapes")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "native", "relay_shapes.cpp"),
           "-L" + PKG, "-Wl,-rpath," + PKG, "-llbp", "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64",
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0 and "relay shapes ok" in r.stdout, (r.stdout, r.stderr[-2000:])
