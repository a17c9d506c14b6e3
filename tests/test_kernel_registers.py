"""No kernel of the library keeps registers in scratch memory: the sizes that the compiler states in the code objects of the built library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2402_15678_amd import build

READELF = next((p for p in (shutil.which("llvm-readelf"), "/opt/rocm/llvm/bin/llvm-readelf") if p and os.path.exists(p)), None)


def _code_objects(lib):
    """gfx950 code objects of the offload bundles in the library (one per translation unit)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = lib.find(magic)
    while at >= 0:
        entries, p = struct.unpack_from("<Q", lib, at + len(magic))[0], at + len(magic) + 8
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", lib, p)
            name = lib[p + 24:p + 24 + n]
            p += 24 + n
            if size and b"gfx950" in name:
                yield lib[at + offset:at + offset + size]
        at = lib.find(magic, at + 1)


@pytest.mark.skipif(READELF is None or not os.path.exists(build.LIB), reason="needs the built library and llvm-readelf")
def test_no_kernel_uses_scratch(tmp_path):
    sizes = {}
    for i, obj in enumerate(_code_objects(open(build.LIB, "rb").read())):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        sizes.update((k, int(v)) for k, v in re.findall(r"\.name: +(_Z\w+)\s+\.private_segment_fixed_size: (\d+)", notes))
    assert len(sizes) > 50
    assert {k: v for k, v in sizes.items() if v} == {}
