"""The machine code of the library's own kernels, read back from the built libisr.so: properties that the kernels rely on
and that neither the compiler nor a run on a GPU would show to be lost."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2108_09413_amd as isr
from paper_2108_09413_amd.build import LIB

LLVM = "/opt/rocm/llvm/bin"


def _parse(listing):
    """{kernel: [(address, instruction, branch target or None)]}"""
    code, base, kernels = None, 0, {}
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if head:
            base, code = int(head.group(1), 16), kernels.setdefault(head.group(2), [])
        elif line.startswith("\t") and code is not None and "//" in line:
            text, _, rest = line.strip().partition("//")
            target = re.search(r"<.*\+0x([0-9a-f]+)>", rest)
            code.append((int(rest.split(":")[0], 16), text.strip(), base + int(target.group(1), 16) if target else None))
    return kernels


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no llvm-objdump")
    isr.lib()
    out = str(tmp_path_factory.mktemp("listing"))
    shutil.copy(LIB, out)
    subprocess.check_call([os.path.join(LLVM, "llvm-objdump"), "--offloading", "libisr.so"], cwd=out, stdout=subprocess.DEVNULL)
    return [os.path.join(out, f) for f in sorted(os.listdir(out)) if f.endswith("gfx950")]


@pytest.fixture(scope="module")
def kernels(code_objects):
    found = {}
    for f in code_objects:
        found.update(_parse(subprocess.check_output([os.path.join(LLVM, "llvm-objdump"), "-d", f], text=True)))
    assert len(found) > 100
    return found


def _open_at_barriers(code):
    """Addresses of the barriers that some path reaches with an LDS access of this wave not known to be complete."""
    index = {a: i for i, (a, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, False)], set()
    while todo:
        i, pending = todo.pop()
        while i < len(code) and (i, pending) not in seen:
            seen.add((i, pending))
            address, text, target = code[i]
            op = text.split()[0]
            if op == "s_barrier" and pending:
                bad.add(address)
            elif op.startswith("ds_"):
                pending = True
            elif op == "s_waitcnt" and "lgkmcnt(0)" in text:
                pending = False
            elif op == "s_endpgm":
                break
            if target is not None and op.startswith("s_cbranch"):
                todo.append((index[target], pending))
            i = index[target] if op == "s_branch" else i + 1
    return bad


def test_a_path_with_an_open_read_is_found():
    def code(wait):
        return [(0, "s_cbranch_scc1 2", 12), (4, "ds_read_b128 v[0:3], v4", None), (8, wait, None), (12, "s_barrier", None), (16, "s_endpgm", None)]
    assert _open_at_barriers(code("s_nop 0")) == {12}
    assert _open_at_barriers(code("s_waitcnt lgkmcnt(1)")) == {12}
    assert _open_at_barriers(code("s_waitcnt lgkmcnt(0)")) == set()


def test_lds_accesses_are_complete_at_every_barrier(kernels):
    """Behind a barrier other waves overwrite what this one has read, with stores or with loads straight into LDS: its reads have to be
    done by then, not only issued, on every path."""
    assert sum(t.startswith("s_barrier") for code in kernels.values() for _, t, _ in code) > 500
    bad = {name: len(at) for name, code in kernels.items() if (at := _open_at_barriers(code))}
    assert not bad


def test_fexpand_stores_are_what_its_waits_count(kernels):
    """fexpand_kernel waits until only what was issued after a step's loads is left, four stores a step of its second kind among it: a
    store that the compiler merged, dropped or moved to another step would let a stage be read before it has landed."""
    checked = 0
    for name, code in kernels.items():
        tiles = re.search(r"fexpand_kernelILi(\d+)E", name)
        if not tiles:
            continue
        steps, stores = [0], {"global_store_dwordx4"}
        for _, text, _ in code:
            op = text.split()[0]
            if op == "s_barrier":
                steps.append(0)
            elif "store" in op and not op.startswith("scratch_"):   # scratch only adds to what is waited for
                stores.add(op)
                steps[-1] += 1
        assert stores == {"global_store_dwordx4"}
        # four steps of the second kind in the loop; behind the last barrier the second layer's result, four stores for 32 channels
        assert steps[-1] == 4 * int(tiles.group(1)) and sorted(n for n in steps[:-1] if n) == [4] * 4, (name, steps)
        checked += 1
    assert checked == 5


def test_expand_and_reduce_stores_are_what_the_waits_count(kernels):
    """The expand-and-reduce kernels of sixteen waves wait until only the stores and loads behind a tile's loads are left: so many stores, in
    both orders of a tile's two halves and of the first tile alone, or behind the last barrier of a tile."""
    wanted = {"proj_expand_reduce_kernel": (3, 2), "expand_reduce256_kernel": (3, 4)}
    checked = 0
    for name, code in kernels.items():
        ops = [t.split()[0] for _, t, _ in code]
        for kernel, (wide, narrow) in wanted.items():
            if kernel in name:
                assert (ops.count("global_store_dwordx4"), ops.count("global_store_dword")) == (wide, narrow), name
                checked += 1
        tile = re.search(r"expand_reduce1024_kernelILi\d+ELi\d+ELi(\d+)E", name)
        if tile:
            n = int(tile.group(1)) // 16
            last = len(ops) - 1 - ops[::-1].index("s_barrier")
            assert (ops[last:].count("global_store_dwordx4"), ops[last:].count("global_store_dword")) == (n, n), name
            assert not any("global_store" in o for o in ops[:last]), name
            checked += 1
        if tile or any(kernel in name for kernel in wanted):
            assert not any("store" in o and not o.startswith("global_store_dword") for o in ops), name
    assert checked == 24


def test_resident_bottleneck_stores_are_what_the_waits_count(kernels):
    """bottleneck_stream_kernel waits until only the four stores behind the next tile's loads are left."""
    checked = 0
    for name, code in kernels.items():
        if "bottleneck_stream_kernel" in name:
            ops = [t.split()[0] for _, t, _ in code]
            stores = [o for o in ops if "store" in o and not o.startswith("scratch_")]   # scratch only adds to what is waited for
            assert sorted(stores) == ["buffer_store_dwordx2"] + 3 * ["buffer_store_dwordx4"], name
            checked += 1
    assert checked == 14


def _is_load_into_lds(text):
    return "load" in text.split()[0] and ("_lds_" in text or text.endswith(" lds"))


def _loads_behind_stores(code):
    """Addresses of the loads into LDS that some path reaches with a store issued since the last barrier."""
    index = {a: i for i, (a, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, False)], set()
    while todo:
        i, stored = todo.pop()
        while i < len(code) and (i, stored) not in seen:
            seen.add((i, stored))
            address, text, target = code[i]
            op = text.split()[0]
            if _is_load_into_lds(text):
                if stored:
                    bad.add(address)
            elif op.startswith(("global_store", "buffer_store")):
                stored = True
            elif op == "s_barrier":
                stored = False
            elif op == "s_endpgm":
                break
            if target is not None and op.startswith("s_cbranch"):
                todo.append((index[target], stored))
            i = index[target] if op == "s_branch" else i + 1
    return bad


def test_a_path_with_a_load_behind_a_store_is_found():
    def code(*ops):
        return [(4 * i, op, 12 if op.startswith("s_cbranch") else None) for i, op in enumerate(ops + ("s_endpgm",))]
    store, load, other = "global_store_dword v0, v1, s[0:1]", "global_load_lds_dwordx4 v[0:1], off", "buffer_load_dwordx4 v0, s[0:3], 0 offen lds"
    assert _loads_behind_stores(code(store, load)) == {4} and _loads_behind_stores(code(store, "s_cbranch_scc1 1", "s_barrier", other)) == {12}
    assert _loads_behind_stores(code(store, "s_barrier", load, other, store)) == set()


def test_loads_into_lds_stand_in_front_of_the_stores_that_the_waits_count(kernels):
    """The kernels that wait until only the stores behind a tile's loads are left: in an interval between two barriers the loads come first.
    (expand_reduce1024_kernel passes its first barrier in all rounds but the first, which has no stores behind it: there what follows the last
    barrier is looked at.)"""
    checked = 0
    for name, code in kernels.items():
        if re.search("proj_expand_reduce_kernel|expand_reduce256_kernel|bottleneck_stream_kernel", name):
            assert sum(_is_load_into_lds(t) for _, t, _ in code) >= 3 and not _loads_behind_stores(code), name
            checked += 1
        elif "expand_reduce1024_kernel" in name:
            texts = [t for _, t, _ in code]
            tail = texts[len(texts) - texts[::-1].index("s_barrier"):]
            loads, stores = [i for i, t in enumerate(tail) if _is_load_into_lds(t)], [i for i, t in enumerate(tail) if t.startswith("global_store")]
            assert loads and max(loads) < min(stores), name
            checked += 1
    assert checked == 38


def test_resident_bottleneck_blocks_keep_to_their_registers(kernels):
    """A reload from scratch waits for the stores and loads in flight: first blocks have none, identity blocks only next to exact halves."""
    scratch = {name: any(t.startswith("scratch_") for _, t, _ in code) for name, code in kernels.items() if "bottleneck_stream_kernel" in name}
    assert len(scratch) == 14
    assert not [name for name, used in scratch.items() if used and not re.search(r"ILb0ELi\d+ELi0E", name)]


def test_stage_kernels_keep_to_their_registers(code_objects):
    """The kernels of the nets on 32 x 32 images, whose rates rest on two to five workgroups a CU with everything in registers."""
    seen = 0
    for f in code_objects:
        notes = subprocess.check_output([os.path.join(LLVM, "llvm-readelf"), "--notes", f], text=True)
        for kernel in notes.split("  - .agpr_count:")[1:]:
            field = {k: re.search(rf"\.{k}:\s+(\S+)", kernel).group(1) for k in ("name", "vgpr_spill_count", "private_segment_fixed_size")}
            if "narrow_" in field["name"] or "short_net" in field["name"]:
                assert (field["vgpr_spill_count"], field["private_segment_fixed_size"]) == ("0", "0"), field
                seen += 1
    assert seen == 10


def test_products_of_the_wide_stages_do_not_wait_for_the_read_in_front(kernels):
    """The pixel operands of the stages of 32 and 64 channels are read steps ahead of their products, in the general form of the
    requantisation as in the others: a product whose wait empties the queue that its own operand was put in last had none ahead."""
    checked = 0
    for name, code in kernels.items():
        if not re.search(r"narrow_kernelILi(64ELi8ELi[26]|32ELi16ELi1)E", name):
            continue
        read = empty = False
        late = products = 0
        for _, text, _ in code:
            op = text.split()[0]
            if op.startswith("ds_read"):
                read, empty = True, False
            elif op == "s_waitcnt" and "lgkmcnt" in text:
                empty = "lgkmcnt(0)" in text
            elif op.startswith("v_mfma"):
                products += 1
                late += read and empty
                read = False
        assert products > 100 and late <= 2, (name, late)
        checked += 1
    assert checked == 3
