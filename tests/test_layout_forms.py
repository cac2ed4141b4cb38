"""The host layout check covers the fused three-way, relay and one-workgroup
kernels and the gathers that idle lanes take part in (native program
tests/native/layout_forms.cpp).  Host only, no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2202_04110_amd", "csrc")


def test_layout_check_covers_every_form(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path / "layout_forms")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(CSRC, "compile.cpp"), os.path.join(CSRC, "hostmem.cpp"),
           os.path.join(ROOT, "tests", "native", "layout_forms.cpp"),
           "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and "layout forms ok" in r.stdout, (r.stdout, r.stderr[-2000:])
