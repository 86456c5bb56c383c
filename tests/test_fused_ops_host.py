"""Which layers share a kernel, by the shifts of their channels (tests/fused_ops_host.cpp)."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import paper_2108_09413_amd as isr
from synth.models import NetBuilder

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2108_09413_amd")
TIE_FREE, TOP, PAIR = 1, 3, 8


@pytest.fixture(scope="module")
def fused_ops(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    isr.lib()   # built
    where = tmp_path_factory.mktemp("fused")
    exe = str(where / "fused_ops_host")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "fused_ops_host.cpp"), os.path.join(PKG, "libisr.so"),
                           f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined", "-o", exe])

    def ops(blob):
        (where / "net.isrm").write_bytes(blob)
        out = subprocess.run([exe, str(where / "net.isrm")], capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stdout + out.stderr
        return [dict(zip(("type", "bneck", "reduce", "form"), map(int, r)))
                for r in re.findall(r"type (-?\d+) bneck (\d+) reduce (\d+) form (-?\d+)", out.stdout)]
    return ops


# shifts below 3 have no top form, a lower clamp above -128 neither that nor pairs
@pytest.mark.parametrize("block,after,fused,form", [
    ("one shift", "one shift", True, PAIR),
    ("one shift", "by channel", True, TOP),
    ("by channel", "one shift", True, TOP),
    ("by channel", "by channel", True, TOP),
    ("shift 2", "one shift", True, PAIR),
    ("shift 2", "by channel", False, PAIR),
    ("one shift", "clamp", False, PAIR),
    ("by channel", "clamp", False, TOP),
    ("clamp", "by channel", True, TIE_FREE),
])
def test_block_and_the_next_stages_first_convolution(fused_ops, block, after, fused, form):
    """The sum of a 64-channel block and the next 1x1 share a kernel unless the block would take a longer form than the top one for it."""
    def kw(kind, c):
        return dict(sh=np.full(c, 2) if kind == "shift 2" else 9 + (np.arange(c) % 3 if kind == "by channel" else np.zeros(c, dtype=np.int64)),
                    zp_out=-100 if kind == "clamp" else -128)
    b = NetBuilder(rng=np.random.default_rng(83), in_shape=(3, 32, 56), num_classes=9)
    t = b.conv(b.conv(b.tensor(3, 32, 56, 0, 74.0), 64, 3, 2, 1, True), 256, 1, 1, 0, True)
    u = b.conv(b.conv(t, 64, 1, 1, 0, True, **kw(block, 64)), 64, 3, 1, 1, True, **kw(block, 64))
    y = b.add(t, b.conv(u, 256, 1, 1, 0, False, sh=kw(block, 256)["sh"]), True)
    u = b.conv(b.conv(y, 128, 1, 1, 0, True, **kw(after, 128)), 128, 3, 1, 1, True)
    t = b.add(b.conv(y, 512, 1, 1, 0, False), b.conv(u, 512, 1, 1, 0, False), True)
    b.fc(b.conv(t, 16, 1, 1, 0, True), 9)
    blocks = [o for o in fused_ops(b.blob()) if o["bneck"] == 2]
    assert [(bool(o["reduce"]), o["form"]) for o in blocks] == [(fused, form)]
