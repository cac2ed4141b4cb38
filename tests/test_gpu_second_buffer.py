"""Graphs whose second message buffer is an option (OR/AND graphs, dense
three-way graphs) still upload, and give the same results, where the device
has room for the graph but not for that buffer.  A native program on the
in-tree liblbp.so refuses allocations above a limit."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2202_04110_amd")


def test_upload_without_the_second_buffer(tmp_path):
    exe = str(tmp_path / "second_buffer")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "native", "second_buffer.cpp"),
           "-L" + PKG, "-Wl,-rpath," + PKG, "-llbp", "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64",
           "-ldl", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0 and "second buffer ok" in r.stdout, (r.stdout, r.stderr[-2000:])
