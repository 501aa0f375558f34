"""What the compiler gave the kernels whose speed hangs on how many wavefronts of them fit a SIMD, as the built library's own
metadata says (no GPU)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2107_13797_amd", "libhaflo.so")
TOOLS = "/opt/rocm/llvm/bin/"


def code_objects(path):
    """The gfx950 code objects of a library's offload bundles."""
    data, at = open(path, "rb").read(), 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(entries):
            offset, size, name_len = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + name_len]
            if b"gfx950" in name and size:
                yield data[at + offset:at + offset + size]
            p += 24 + name_len
        at += len(magic)


@pytest.fixture(scope="module")
def vector_registers(tmp_path_factory):
    """Kernel's mangled name -> vector registers of a lane."""
    if not os.path.exists(LIB) or not shutil.which(TOOLS + "llvm-readelf"):
        pytest.skip("no built library, or no tool to read its notes")
    out = {}
    for i, obj in enumerate(code_objects(LIB)):
        path = str(tmp_path_factory.mktemp("co") / ("%d.co" % i))
        open(path, "wb").write(obj)
        notes = subprocess.run([TOOLS + "llvm-readelf", "--notes", path], capture_output=True, text=True, check=True).stdout
        for name, count in re.findall(r"\.name:\s+(_Z\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", notes):
            out[name] = int(count)
    assert out
    return out


def test_two_blocks_of_the_single_form_share_a_compute_unit(vector_registers):
    """k_rns_group of 1024-bit moduli in the single form: the launch counts on two blocks of nine wavefronts to a compute unit,
    which is six to one of its SIMDs, 512 / 6 registers each in steps of eight (with 88 of them the second block waits: the key
    owner's 3000 encryptions at a 2048-bit key took 3.20 instead of 2.99 ms)."""
    found = [v for k, v in vector_registers.items() if re.search(r"k_rns_groupILi10ELi1ELi9ELi1ELi0ELb0ELb0EE", k)]
    assert len(found) == 1 and found[0] <= 80
