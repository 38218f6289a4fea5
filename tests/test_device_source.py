"""Properties of the device sources that no result shows."""
import glob
import os
import re
import struct
import subprocess

import pytest

from paper_2606_18431_amd import build, tas

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2606_18431_amd", "csrc")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))),
                         ids=os.path.basename)
def test_inline_assembly_holds_no_instruction(path):
    """The compiler separates dependent instructions by the wait states the
    chip needs (a vector instruction after a lane read of its scalar operand
    needs two), but not where one of them is inline assembly text. Assembly
    statements here only constrain registers; an asm label names an LLVM
    intrinsic, which the compiler schedules like any other instruction."""
    src = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(path).read(), flags=re.S)
    texts = re.findall(r"\b(?:__asm__|__asm|asm)\b[^(]*\(\s*((?:\"[^\"]*\"\s*)+)", src)
    assert len(texts) == len(re.findall(r"\b(?:__asm__|__asm|asm)\b", src))
    for t in texts:
        t = "".join(re.findall(r"\"([^\"]*)\"", t))
        assert t == "" or t.startswith("llvm.amdgcn."), t


def kernels(path, tmp_path):
    """{kernel: vector registers} of the gfx950 code objects in a library."""
    data = open(path, "rb").read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", {}
    for m in re.finditer(magic, data):
        at = m.end()
        n, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if not name.endswith("gfx950") or not size:
                continue
            obj = tmp_path / "code.o"
            obj.write_bytes(data[m.start() + off:m.start() + off + size])
            readelf = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin",
                                   "llvm-readelf")
            notes = subprocess.check_output([readelf, "--notes", str(obj)], text=True)
            for k in re.split(r"\n\s*- \.agpr_count", notes)[1:]:
                out[re.search(r"\.name:\s+(\S+)", k).group(1)] = \
                    int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1))
    return out


def test_simulator_builds_leave_room_for_four_waves(tmp_path):
    """Every single-server build fits four waves a SIMD (128 vector registers
    each), which is what the LDS holds at 64 sequences."""
    found = {k: v for k, v in kernels(tas.LIB_PATH, tmp_path).items() if "sim_kernel" in k}
    assert len(found) == 8, found
    assert all(v <= 128 for v in found.values()), found
