"""Host launchers of libffth.so called for shapes without a kernel (no GPU)."""
import os
import shutil
import subprocess

import pytest

from paper_1712_05145_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(build.LIB), reason="no host compiler or library")
def test_grouped_launchers_refuse_shapes_without_a_kernel(tmp_path):
    exe = str(tmp_path / "launch_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_1712_05145_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_check.cpp"), build.LIB,
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "OK" in out.stdout, out.stdout + out.stderr
