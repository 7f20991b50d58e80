"""What the compiler gave the kernels of the built library: none of them keeps registers in scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2603_02731_amd as mx
from paper_2603_02731_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """The gfx950 code objects of the library, one per source file."""
    mx.lib()
    with open(build.LIB, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if name.endswith("gfx950"):
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def test_no_kernel_spills(tmp_path):
    hipcc = shutil.which(build.HIPCC)
    near = [os.path.join(os.path.dirname(os.path.realpath(hipcc)), d, "llvm-readelf") for d in (".", "../llvm/bin", "../lib/llvm/bin")] \
        if hipcc else []
    readelf = next((p for p in near if os.path.exists(p)), shutil.which("llvm-readelf"))
    if readelf is None:
        pytest.skip("no llvm-readelf beside the compiler")
    scratch = {}
    for i, code in enumerate(code_objects()):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([readelf, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        sizes = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
        names = re.findall(r"\.symbol:\s+(\S+)\.kd", notes)
        assert len(sizes) == len(names)
        scratch.update(zip(names, map(int, sizes)))
    assert len(scratch) >= 25 and sum("owner_kernel" in n for n in scratch) == 4, sorted(scratch)
    spilled = {n: s for n, s in scratch.items() if s}
    assert not spilled, f"bytes of scratch per lane: {spilled}"
