"""The linear that keeps the rows of x in registers does keep them there: no variant of it spills.  Read from the
resource notes of the built library's own code objects."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2604_16498_amd import build

READELF = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin", "llvm-readelf")


def code_objects(path):
    data, at = open(path, "rb").read(), 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + length]:
                yield data[at + off:at + off + size]
            entry += 24 + length
        at += 24


def test_no_variant_spills(tmp_path):
    tool = READELF if os.path.exists(READELF) else shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin")
    if tool is None:
        pytest.skip("no llvm-readelf beside hipcc")
    seen, spilled = 0, []
    for i, co in enumerate(code_objects(build.LIB)):
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(co)
        notes = subprocess.run([tool, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name: +(\S+)", kernel)[1]
            if "gemm_bf16_rows_kernel" in name:
                seen += 1
                if re.search(r"(vgpr_spill_count|private_segment_fixed_size): +[1-9]", kernel):
                    spilled.append(name)
    assert seen > 50 and not spilled, spilled
