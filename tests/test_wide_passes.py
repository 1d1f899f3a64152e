"""The passes of calls of more than 64 tokens stay inside the workspace: the library's own host
arithmetic, swept on the CPU by a small driver linked to it."""
import os
import shutil
import subprocess

import pytest

from paper_2609_31975_amd import build, ffn

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_pass_fits_the_workspace(tmp_path):
    ffn.lib()
    exe = str(tmp_path / "wide_passes")
    csrc = os.path.join(build.PKG, "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", csrc, "-I", os.path.join(build.ROOT, "include"),
                    "-I", "/opt/rocm/include", os.path.join(HERE, "wide_passes_driver.cpp"), build.LIB,
                    "-L/opt/rocm/lib", "-lamdhip64", f"-Wl,-rpath,{build.PKG}", "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    calls, passes = map(int, res.stdout.split())
    assert calls > 400000 and passes > calls  # the sweep did reach the path
