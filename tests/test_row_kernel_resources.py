"""LDS and scratch of the compiled row kernels, read from the library's own gfx950 code
objects: the fixed LDS is the point lists the planner counts, or nothing, and no row is
kept in scratch."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1509_04394_amd import build, fz

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    """The AMDGPU ELF images inside the library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:  # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, num = struct.unpack_from("<HH", data, at + 58)
            yield data[at:at + shoff + size * num]
        at = data.find(b"\x7fELF", at + 4)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    fz.lib()
    found, path = {}, str(tmp_path_factory.mktemp("co") / "co")
    for image in code_objects(build.LIB):
        with open(path, "wb") as f:
            f.write(image)
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        for k in notes.split("- .agpr_count")[1:]:
            value = lambda name: re.search(rf"\.{name}:\s+(\S+)", k).group(1)
            symbol = [n for n in re.findall(r"\.name:\s+(\S+)", k) if n.startswith("_Z")][0]
            found[symbol] = int(value("group_segment_fixed_size")), int(value("private_segment_fixed_size"))
    assert len(found) > 100
    return found


def test_row_kernels_hold_what_the_planner_counts(kernels):
    lists = {2: 4 * (256 * 4 + 32) + 8, 3: 4 * (256 * 5 + 32) + 8}
    seen = 0
    for name, (lds, scratch) in kernels.items():
        if m := re.match(r"_ZN2fz8k_rowgenILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb([01])E", name):
            assert lds == (lists[int(m[4])] if m[5] == "1" else 0) and scratch == 0, (name, lds, scratch)
        elif m := re.match(r"_ZN2fz\d+k_rowfuse(_direct|_batch)?ILi(\d)E", name):
            # the gray kernels' six wavefronts a SIMD take two or three registers to scratch
            assert lds == (0 if m[1] == "_direct" else lists[int(m[2])]) and scratch <= 12, (name, lds, scratch)
        else:
            continue
        seen += 1
    assert seen >= 40
