"""Registers of the built kernels, read from their code objects' notes: the compiler
flag that keeps the pair kernel's loops from spilling does so only as long as the
compiler heeds it, and nothing else would show that it stopped."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2405_04463_amd", "_build")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(source, folder):
    """{kernel: (VGPRs spilled, scratch bytes)} of the gfx950 code of an object of the build."""
    obj = os.path.join(BUILD, source + ".o")
    if not (os.path.exists(obj) and (os.path.exists(READELF) or shutil.which("llvm-readelf"))):
        pytest.skip("no built object, or no reader")
    data = open(obj, "rb").read()
    at = data.index(MAGIC)
    count, = struct.unpack_from("<Q", data, at + len(MAGIC))
    pos = at + len(MAGIC) + 8
    for _ in range(count):
        off, size, idlen = struct.unpack_from("<QQQ", data, pos)
        name = data[pos + 24:pos + 24 + idlen].decode()
        pos += 24 + idlen
        if "gfx950" in name:
            elf = os.path.join(folder, source + ".co")
            with open(elf, "wb") as f:
                f.write(data[at + off:at + off + size])
    tool = READELF if os.path.exists(READELF) else "llvm-readelf"
    notes = subprocess.run([tool, "--notes", elf], capture_output=True, text=True, check=True).stdout
    out = {}
    for part in notes.split("  - .agpr_count:")[1:]:
        get = lambda key: re.search(rf"\.{key}:\s+(\S+)", part).group(1)  # noqa: E731
        out[get("name")] = (int(get("vgpr_spill_count")), int(get("private_segment_fixed_size")))
    return out


def test_pair_kernel_spills(tmp_path):
    found = {k: v for k, v in kernels("pair_dot.hip", str(tmp_path)).items() if "pair_dot_kernel" in k}
    assert len(found) == 2
    # 27 and 28 with the flag, 63 and 78 without, 41 and 45 of the instructions in the loops
    assert all(spilled <= 32 and scratch <= 128 for spilled, scratch in found.values()), found


def test_rotation_kernels_do_not_spill(tmp_path):
    for source, name in (("rot_dot.hip", "rot_dot_kernel"), ("rot_dot.hip", "rot_dot_split_kernel"),
                         ("dot32.hip", "rot_dot32_kernel")):
        found = {k: v for k, v in kernels(source, str(tmp_path)).items() if name in k}
        assert found and all(spilled == 0 for spilled, _ in found.values()), found
