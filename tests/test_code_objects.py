"""CPU: the gfx950 code of the built library, disassembled."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_26762_amd import protokv as pk

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The library's gfx950 code objects, as files."""
    if not (os.path.exists(OBJDUMP) and os.path.exists(READELF)):
        pytest.skip("no LLVM tools")
    d = tmp_path_factory.mktemp("code")
    so = shutil.copy(pk.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", so], cwd=d, check=True, capture_output=True)
    return sorted(d.glob("*gfx950*"))


@pytest.fixture(scope="module")
def kernels(objects):
    """{mangled name: instructions} of every kernel."""
    out = {}
    for f in objects:
        text = subprocess.run([OBJDUMP, "-d", f], check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\w+)>:\n((?:\t.*\n)+)", text, re.M):
            out[name] = [l.split("//")[0].strip() for l in body.splitlines()]
    assert out
    return out


def test_maintenance_reads_lanes_with_all_lanes_active(kernels):
    """The merge scan reads a slot's filter dims from the lanes that hold them.
    A register that a divergent branch copies or reloads is written in the
    active lanes only, so those reads stand outside every such branch: the last
    write of exec before them does not narrow it.  (Reads of the registers that
    v_writelane fills are scalar spills and read no other lane's value.)"""
    found = 0
    for name, code in kernels.items():
        if "k_maintain" not in name:
            continue
        spill = {m.group(1) for l in code if (m := re.match(r"v_writelane_b32 (v\d+),", l))}
        last = ""
        for l in code:
            if re.match(r"s_\w+ exec,|s_\w*saveexec", l):
                last = l
            m = re.match(r"v_readlane_b32 s\d+, (v\d+), \d+", l)
            if m and m.group(1) not in spill:
                found += 1
                assert "and_saveexec" not in last, f"{name}: {l} after {last}"
    assert found >= 6 * 8   # six kernels, at least four dims of K and of V


def test_descriptors_are_aligned_kernel_arguments(objects):
    """A launch whose frame descriptor (sid, slot, ... of 64 streams) lies 8 bytes
    off a multiple of 16 takes 0.13 us longer.  The readout's descriptor, 80 bytes,
    comes behind the workspace without padding: its launches pay for the bytes."""
    frames = readouts = 0
    for f in objects:
        notes = subprocess.run([READELF, "--notes", f], check=True, capture_output=True, text=True).stdout
        for args in re.findall(r"\.args:\n(.*?)(?=\n    \.\w)", notes, re.S):
            structs = [(int(o), int(n)) for o, n in re.findall(
                r"\.offset: +(\d+)\s+\.size: +(\d+)\s+\.value_kind: +by_value", args) if int(n) > 16]
            for offset, size in structs[2:]:   # behind Dims and Workspace
                if size > 256:
                    frames += 1
                    assert offset % 16 == 0, (f.name, structs)
                else:
                    readouts += 1
                    assert offset == sum(structs[1]), (f.name, structs)
    assert frames >= 12 and readouts >= 6
