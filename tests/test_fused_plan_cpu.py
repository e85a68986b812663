"""The plan of the fused pass over B on devices of 1 to 304 compute units
(tests/fused_plan_driver.cpp, host code of libsdp only)."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1707_05058_amd")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_members_have_units_and_tiles_cover(tmp_path):
    exe = str(tmp_path / "fused_plan_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(PKG, "csrc"), "-I", "/opt/rocm/include",
                    os.path.join(HERE, "fused_plan_driver.cpp"), "-o", exe, "-L", PKG, "-l:libsdp.so",
                    "-L", "/opt/rocm/lib", "-lamdhip64", f"-Wl,-rpath,{PKG}:/opt/rocm/lib"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(re.match(r"(\d+) plans", r.stdout).group(1)) > 100
