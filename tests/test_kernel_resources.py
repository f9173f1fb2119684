"""What the built kernels take, from the metadata of the library's own code
objects: no whole-map kernel of batches with per-pair lengths, thresholds or
offsets keeps a lane's words in scratch memory."""
from __future__ import annotations

import os
import re
import struct
import subprocess

import pytest

import paper_1910_03936_amd as paf

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    with open(path, "rb") as f:
        lib = f.read()
    at = lib.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", lib, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", lib, pos)
            name = lib[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in name and size:
                yield lib[at + off:at + off + size]
        at = lib.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Mangled kernel name -> bytes of scratch a lane has."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    paf.load_library()
    out = {}
    for i, co in enumerate(_code_objects(os.path.join(os.path.dirname(paf.__file__), "libpaf.so"))):
        p = tmp_path_factory.mktemp("co") / f"{i}.elf"
        p.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True, check=True).stdout
        for k in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name: +(\S+)", k).group(1)
            out[name] = int(re.search(r"\.private_segment_fixed_size: +(\d+)", k).group(1))
    return out


def test_general_whole_map_kernels_without_scratch(scratch):
    # (mangled: whole_kernel<EMAX, GENERAL, FS>)
    general = {k: v for k, v in scratch.items() if re.search(r"whole_kernelILi\d+ELb1E", k)}
    assert len(general) % 15 == 0 and general   # one per threshold class and mask
    assert {k: v for k, v in general.items() if v} == {}
