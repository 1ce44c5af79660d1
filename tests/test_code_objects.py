"""What the compiler made of the kernels, read from the notes of the library's own code objects."""
import os
import re
import struct
import subprocess

import pytest

from paper_2410_16179_amd import binding as mp

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: {note field: number}} of every gfx950 code object in the built library."""
    tmp = tmp_path_factory.mktemp("code_objects")
    fat = str(tmp / "fat")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", f".hip_fatbin={fat}", mp.LIB_PATH, str(tmp / "rest")], check=True)
    data = open(fat, "rb").read()
    got = {}
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):    # one bundle per source file
        at = m.end()
        count = struct.unpack_from("<Q", data, at)[0]
        at += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" not in target or not size:
                continue
            path = str(tmp / f"{m.start()}.elf")
            open(path, "wb").write(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, capture_output=True, text=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                name = re.search(r"^    \.name:\s+(\S+)", part, re.M).group(1)
                got[name] = {k: int(v) for k, v in re.findall(r"^    \.(\w+):\s+(\d+)$", part, re.M)}
    assert got
    return got


def test_keys_of_float32_hashing_are_staged_on_16_byte_boundaries(kernels):
    # the block whose size the launch gives begins where the fixed part ends; its rows are read 16 bytes at a time
    sizes = [v["group_segment_fixed_size"] for k, v in kernels.items() if "hash_keys_f32_kernel" in k]
    assert len(sizes) == 2 and all(s % 16 == 0 for s in sizes), sizes


def test_gather_takes_lds_by_the_heads_of_its_workgroup(kernels):
    # index lists for eight heads in a workgroup of one wavefront leave room for nine of sixteen wavefronts
    sizes = [v["group_segment_fixed_size"] for k, v in kernels.items() if "gather_estimate_kernel" in k]
    assert sizes and all(s == 0 for s in sizes), sizes
