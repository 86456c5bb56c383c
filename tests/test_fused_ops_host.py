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
        return [{k: int(v) for k, v in re.findall(r"(\w+) (-?\d+)", line)} for line in out.stdout.splitlines()]
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


# halves of a multiplier (odd) * 2^tz lie (odd) / 2 steps and more from zero, its accumulators 2^(30 + shift - tz) and more
@pytest.mark.parametrize("tz,sh,zp,relu,free", [
    (29, 9, -128, True, True), (29, 9, 100, True, True), (29, 9, -128, False, True), (29, 9, -126, False, False), (29, 9, 0, False, False),
    (18, 9, 127, False, True), (21, 9, 127, False, True), (22, 9, 127, False, False), (22, 9, 0, False, True), (22, 22, 127, False, True),
    (30, 9, -127, False, False), (30, 9, -128, False, True),
])
def test_halves_that_no_clamp_hides(fused_ops, tz, sh, zp, relu, free):
    b = NetBuilder(rng=np.random.default_rng(84), in_shape=(3, 8, 8), num_classes=9)
    t = b.conv(b.tensor(3, 8, 8, 0, 74.0), 64, 3, 1, 1, True)
    odd = ((1 << 30) >> tz) + (1 if tz < 30 else 0)          # the fewest steps
    t = b.conv(t, 256, 1, 1, 0, relu, m0=np.full(256, odd << tz), sh=np.full(256, sh), zp_out=zp)
    b.fc(b.conv(t, 16, 1, 1, 0, True), 9)
    assert [bool(o["tie_free"]) for o in fused_ops(b.blob()) if o["cout"] == 256] == [free]


@pytest.mark.parametrize("relu,ma,mb,free", [(True, 1 << 19, 1 << 19, True), (False, 1 << 19, 1 << 19, False), (False, 700001, 800003, True), (True, -(1 << 19), 1 << 19, True)])
def test_halves_in_an_add_that_no_clamp_hides(fused_ops, relu, ma, mb, free):
    b = NetBuilder(rng=np.random.default_rng(85), in_shape=(3, 8, 8), num_classes=9)
    t = b.conv(b.conv(b.tensor(3, 8, 8, 0, 74.0), 64, 3, 1, 1, True), 192, 1, 1, 0, True)
    u = b.conv(b.conv(t, 64, 3, 1, 1, True), 192, 1, 1, 0, False)
    b.fc(b.conv(b.add(t, u, relu, ma=ma, mb=mb, sh=20, zp_out=-7), 16, 1, 1, 0, True), 9)
    assert [bool(o["add_tie_free"]) for o in fused_ops(b.blob()) if o["add_tie_free"] >= 0] == [free]


class _Blob(Exception):
    pass


class _Recorder:
    """Stands for the library in a test that builds a net and loads it."""

    def isr_load_model(self, blob):
        raise _Blob(blob)


def _kernel(o):
    if o["stem"]:
        return "first layer with pooling"
    if o["bneck"]:
        return {1: "bottleneck head", 2: "bottleneck block", 4: "bottleneck block with projection"}[o["bneck"]] + (" and next" if o["reduce"] else "")
    if o["xr"]:
        return f"expand {o['cout']} reduce {o['next']}"
    if (o["k"], o["stride"]) == (3, 1) and o["cout"] in (128, 256, 512):
        return f"staged rows {128 if o['cout'] == 128 else 256}"
    return "other"


# what the GPU tests of these names run in the top-byte form, and the first layer's in pairs
@pytest.mark.parametrize("test,args,form,kernels", [
    ("test_first_layer_with_pooling_in_the_short_forms", ((37, 28), "pairs"), PAIR, {"first layer with pooling"}),
    ("test_first_layer_with_pooling_in_the_short_forms", ((37, 28), "top byte"), TOP, {"first layer with pooling"}),
    ("test_top_form_in_bottleneck_heads", (256,), TOP, {"bottleneck head"}),
    ("test_top_form_in_bottleneck_blocks", ((30, 20),), TOP, {"bottleneck block", "bottleneck block with projection"}),
    ("test_top_form_in_a_block_with_the_next_stages_first_convolution", ((32, 56), 2, 2, "_TopForm"), TOP, {"bottleneck block and next"}),
    ("test_top_form_in_a_block_with_the_next_stages_first_convolution", ((32, 56), 2, 2, "_NextByChannel"), TOP, {"bottleneck block and next"}),
    ("test_top_form_in_staged_rows_of_256_channels", (9,), TOP, {"staged rows 256"}),
    ("test_top_form_in_staged_rows_against_the_oracle", ((10, 4), 2, 1), TOP, {"staged rows 128", "staged rows 256"}),
    ("test_top_form_in_expand_add_and_next_reduce", (), TOP, {"expand 512 reduce 128", "expand 512 reduce 256", "expand 1024 reduce 256"}),
])
def test_forms_that_the_gpu_tests_run(fused_ops, monkeypatch, test, args, form, kernels):
    """Where the planner prefers another form, a test of one that is still in use would silently run the other."""
    import test_gpu_parity as gpu

    def builder(cls):
        monkeypatch.setattr(gpu, "NetBuilder", cls)
    args = [getattr(gpu, a) if isinstance(a, str) and hasattr(gpu, a) else a for a in args]
    f = getattr(gpu, test)
    with pytest.raises(_Blob) as net:
        f(_Recorder(), *([builder] if "builder" in f.__code__.co_varnames[:2] else []), *args)
    assert kernels <= {_kernel(o) for o in fused_ops(net.value.args[0]) if o["form"] == form}
