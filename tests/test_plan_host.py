"""Where the planner's tensors lie while ops of different images run side by side (tests/plan_host.cpp)."""
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


def three_stages(last, first="3x3"):
    """A net on 32x32 images whose last stage ends in `last`; the first layer as the stage kernels take it or, 5x5, on its own."""
    b = NetBuilder(rng=np.random.default_rng(94), in_shape=(3, 32, 32), num_classes=7)
    k = int(first[0])
    t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, k, 1, k // 2, True)
    for ch in (16, 32, 64):
        if ch > 16:
            u = b.conv(b.conv(t, ch, 3, 2, 1, True), ch, 3, 1, 1, False)
            t = b.add(b.conv(t, ch, 1, 2, 0, False), u, True)
        t = b.add(t, b.conv(b.conv(t, ch, 3, 1, 1, True), ch, 3, 1, 1, False), True)
    if last == "pooling":
        t = b.gap(t)
    elif last == "max pooling":
        t = b.maxpool(t, 2, 2, 0)
    elif last == "convolution":
        t = b.gap(b.conv(t, 80, 3, 1, 1, True))
    b.fc(t, 7)
    return b.blob()


@pytest.fixture(scope="module")
def plan_host(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    isr.lib()   # built
    exe = str(tmp_path_factory.mktemp("plan") / "plan_host")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "plan_host.cpp"), os.path.join(PKG, "libisr.so"),
                           f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined", "-o", exe])
    return exe


@pytest.mark.parametrize("first", ["3x3", "5x5"])
@pytest.mark.parametrize("last", ["pooling", "max pooling", "convolution", "nothing"])
def test_stages_of_different_images_lie_apart(plan_host, tmp_path, last, first):
    """The three stages share a launch, in which images are at different stages, only where no stage's result lies over what
    another image still reads: not where the last stage stores its result, in the space of the first one's."""
    blob = tmp_path / "net.isrm"
    blob.write_bytes(three_stages(last, first))
    out = subprocess.run([plan_host, str(blob)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    rows = [dict(zip(("copies", "narrow", "head", "apart", "by_bytes"), r))
            for r in re.findall(r"copies (\d+) narrow (\d+ \d+ \d+) head (\d) apart (\d) by_bytes (\d)", out.stdout)]
    stages = [r for r in rows if r["narrow"] == "16 32 64"]
    assert len(stages) == 4   # numbers of copies
    for r in rows:
        # (overlaps in the padding behind the last image count as well: never apart in word only)
        assert r["apart"] <= r["by_bytes"], r
    for r in stages:
        assert (r["head"] == "1") == (last == "pooling")
        if last == "pooling":
            assert r["apart"] == "1", r
        elif int(r["copies"]) > 1:
            assert r["apart"] == r["by_bytes"] == "0", r


@pytest.mark.gpu
@pytest.mark.parametrize("last,first,together", [("max pooling", "3x3", False), ("convolution", "3x3", False), ("nothing", "5x5", False), ("pooling", "5x5", True)])
def test_stages_whose_result_is_stored_run_in_launches_of_their_own(last, first, together):
    """256 copies against the op-by-op kernels; with a 5x5 first layer the first stage reads its input from memory."""
    print(f"{first} first layer, three stages, then {last}", flush=True)
    m = isr.isr_load_model(three_stages(last, first))
    isr.isr_set_workspace(m, 256)
    x = np.random.default_rng(13).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    isr.isr_profile(m, 1)
    fused = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, 256)
    names = [k["name"] for k in isr.isr_profile_read(m)]
    assert [sum(n.startswith(k) for n in names) for k in ("narrow_kernel", "narrow_chain_kernel")] == ([0, 1] if together else [3, 0]), names
    isr.isr_set_fusion(m, 0)
    for a, b in zip(fused, isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, 256)):
        assert np.array_equal(a, b)
    m.close()
