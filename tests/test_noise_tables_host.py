"""The sampler's tables of every sigma on the host: tests/noise_tables_host.cpp reads them as the kernels do, around
every threshold and bucket edge, and times their construction against that of the thresholds they hold."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_09413_amd", "csrc")


def test_tables_of_every_sigma(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "noise_tables_host")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, os.path.join(ROOT, "tests", "noise_tables_host.cpp"), os.path.join(CSRC, "noise_table.cpp"), "-o", exe])
    proc = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert proc.returncode == 0, proc.stdout
    assert int(re.search(r"checked (\d+)", proc.stdout).group(1)) > 10_000_000
    cost = {s: (float(p), float(b)) for s, p, b in re.findall(r"sigma (\d+) pixel (\S+) stored (\S+)", proc.stdout)}
    # shares of the time that the thresholds take: 0.08 for the pixels' table of sigma 256 and 0.4 for the stored-noise one
    # of sigma 1000 when each is filled once; filled shape by shape until one fits, 0.6 and 1.6
    assert cost["256"][0] < 0.3 and cost["1000"][1] < 0.8, cost
