"""The round kernel of the sketches runs once per task, most of them of a few
arcs: registers it spills to scratch are stored and read for every one of them."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_1503_03635_amd.build as b

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
EM_AMDGPU = 224


def _code_objects(blob):
    """The gfx950 ELF images embedded in the library."""
    at = blob.find(b"\x7fELF", 4)
    while at >= 0:
        machine, = struct.unpack_from("<H", blob, at + 18)
        if machine == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            entsize, num = struct.unpack_from("<HH", blob, at + 58)
            yield blob[at:at + shoff + entsize * num]
        at = blob.find(b"\x7fELF", at + 4)


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """Spilled vector registers of every kernel of the library."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(b.LIB):
        b.build()
    out = {}
    with open(b.LIB, "rb") as f:
        blob = f.read()
    path = tmp_path_factory.mktemp("co") / "co.elf"
    for image in _code_objects(blob):
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"^\s+\.name:\s+(_Z\S*k_\S+)$", notes, re.M)
        counts = re.findall(r"^\s+\.vgpr_spill_count:\s+(\d+)$", notes, re.M)
        assert len(names) == len(counts)
        out.update(zip(names, map(int, counts)))
    return out


def test_round_kernel_keeps_its_registers(spills):
    tasks = {name: n for name, n in spills.items() if "k_ads_tasks" in name}
    assert len(tasks) == 6, sorted(spills)
    assert max(tasks.values()) <= 8, tasks
