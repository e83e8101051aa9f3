"""CPU: what the compiler states about the built library's kernels: no kernel keeps registers in scratch memory (spills), but for one whose
figures stand beside its rule (the two-tile form for several index widths, whose 4-bit part does)."""
import shutil
import re
import struct
import subprocess
from pathlib import Path

import pytest

from paper_2506_12038_amd.build import LIB

READELF = Path("/opt/rocm/llvm/bin/llvm-readelf")
KNOWN = {"gemv_tokens_mixed_kernel<2, 16, 8, false>"}


def _code_objects(data):
    """The gfx950 code objects of every offload bundle in the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in triple and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


@pytest.mark.skipif(not READELF.exists() or shutil.which("c++filt") is None, reason="no llvm-readelf or c++filt")
def test_no_kernel_spills(tmp_path):
    kernels, spilling = 0, set()
    for i, code in enumerate(_code_objects(LIB.read_bytes())):
        f = tmp_path / f"{i}.co"
        f.write_bytes(code)
        notes = subprocess.run([str(READELF), "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for name, scratch in re.findall(r"^\s+\.name:\s+(_ZN3lcd\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", notes, flags=re.M):
            kernels += 1
            if int(scratch):
                text = subprocess.run(["c++filt", name], capture_output=True, text=True, check=True).stdout
                spilling.add(re.sub(r"^void ", "", text.replace("lcd::", "")).split("(")[0])
    assert kernels > 200
    assert spilling <= KNOWN, spilling - KNOWN
