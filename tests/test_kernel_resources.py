"""Registers of the built kernels, from the code object metadata of the built library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1508_05610_amd", "liblf2.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(READELF),
                                reason="needs the built library and llvm-readelf")


def _code_objects():
    """The gfx950 code objects of the library's offload bundles."""
    with open(LIB, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            pos += 24
            if b"gfx950" in data[pos:pos + idlen] and size:
                yield data[at + off:at + off + size]
            pos += idlen
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (VGPRs, spilled VGPRs, scratch bytes a lane)}"""
    out = {}
    path = str(tmp_path_factory.mktemp("co") / "kernels.co")
    for co in _code_objects():
        with open(path, "wb") as f:
            f.write(co)
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True,
                               check=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\n\s+\.name:\s+(\S+)", k).group(1)
            out[name] = tuple(int(re.search(rf"\n\s+\.{f}:\s+(\d+)", k).group(1))
                              for f in ("vgpr_count", "vgpr_spill_count",
                                        "private_segment_fixed_size"))
    return out


def test_transposing_tiles_leave_room_for_their_blocks(kernels):
    """Where three blocks of a transposing z tile fit a CU's LDS (at most 160 / 3 KB
    with its twiddles), their registers do as well from 48 points on (six waves a SIMD
    of 512 registers: at most 80), 384 and 768 points excepted; and no tile spills."""
    seen = set()
    for name, (vgprs, spills, scratch) in kernels.items():
        m = re.fullmatch(r"_ZN3lf211k_strided_tILi(\d+)ELin?1EEEvNS_5SArgsE", name)
        if not m:
            continue
        n = int(m.group(1))
        seen.add(n)
        assert spills == 0 and scratch == 0, (name, vgprs, spills, scratch)
        cols = 64 if n <= 128 else 32 if n <= 256 else 16 if n <= 512 else 8 if n <= 1024 else 4
        if n >= 48 and n not in (384, 768) and 8 * n * (cols + 1) <= 160 * 1024 // 3:
            assert vgprs <= 80, (name, vgprs)
    assert {16, 96, 192, 320, 640, 1024} <= seen
