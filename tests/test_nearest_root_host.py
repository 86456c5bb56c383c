"""The correction of the sampler's binary32 root (tests/nearest_root_host.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_root_of_every_mantissa(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "nearest_root_host")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_2108_09413_amd", "csrc"), os.path.join(ROOT, "tests", "nearest_root_host.cpp"), "-o", exe])
    proc = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert proc.returncode == 0, proc.stdout
    assert proc.stdout.split() == ["checked", str(3 * 3 << 24)]
