"""No kernel of the built library keeps registers in scratch memory: every ring
and stage of the marches is meant to stay in registers.  Read from the metadata
of the library's own code objects; nothing runs on a GPU."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2404_02813_amd", "librsf.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 ELF images of the library's offload bundles."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, p - 8)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n].decode()
            p += 24 + n
            if "gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def test_no_kernel_uses_scratch(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("needs the built library and llvm-readelf")
    scratch = {}
    for k, image in enumerate(code_objects(LIB)):
        path = tmp_path / f"{k}.co"
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        sizes = re.findall(r"\.private_segment_fixed_size:\s*(\d+)", notes)
        names = re.findall(r"\.symbol:\s*'?(\S+?)\.kd", notes)
        assert len(sizes) == len(names)
        scratch.update(zip(names, map(int, sizes)))
    assert len(scratch) > 500
    spilled = {n: s for n, s in scratch.items() if s}
    assert not spilled
