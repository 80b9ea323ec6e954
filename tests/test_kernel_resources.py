"""Registers and load sequences of the built kernels, from the code objects of the built
library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1508_05610_amd", "liblf2.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(
    not all(os.path.exists(f) for f in (LIB, READELF, OBJDUMP)),
    reason="needs the built library, llvm-readelf and llvm-objdump")


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
    of 512 registers: at most 80), 384 points excepted; and no tile spills."""
    seen = set()
    for name, (vgprs, spills, scratch) in kernels.items():
        m = re.fullmatch(r"_ZN3lf211k_strided_tILi(\d+)ELin?1EEEvNS_5SArgsE", name)
        if not m:
            continue
        n = int(m.group(1))
        seen.add(n)
        assert spills == 0 and scratch == 0, (name, vgprs, spills, scratch)
        cols = 64 if n <= 128 else 32 if n <= 256 else 16 if n <= 512 else 8 if n <= 1024 else 4
        if n >= 48 and n != 384 and 8 * n * (cols + 1) <= 160 * 1024 // 3:
            assert vgprs <= 80, (name, vgprs)
    assert {16, 96, 192, 320, 640, 1024} <= seen


def _waits_among_loads(code):
    """Waits for global loads between one load and the next, nothing being stored to LDS,
    met at a barrier or computed between the two."""
    n, waited, loading = 0, False, False
    for line in code.splitlines():
        op = line.split()[0] if line.startswith("\t") and line.split() else ""
        if op.startswith("global_load"):
            n += waited and loading
            loading, waited = True, False
        elif op == "s_waitcnt" and "vmcnt" in line:
            waited = True
        elif op.startswith(("ds_write", "s_barrier", "global_store", "v_fma", "v_add_f", "v_mul_f",
                            "v_sub_f")):
            loading = waited = False
    return n


def _kernel_waits(mangled, tmp_path):
    path = str(tmp_path / "kernels.co")
    for co in _code_objects():
        if mangled.encode() not in co:
            continue
        with open(path, "wb") as f:
            f.write(co)
        code = subprocess.run([OBJDUMP, f"--disassemble-symbols={mangled}", path],
                              capture_output=True, text=True, check=True).stdout
        assert "global_load" in code
        return _waits_among_loads(code)
    raise AssertionError(f"no kernel {mangled}")


# complex x passes of one and of many stages, one component (backward) and several;
# real ones of interleaved components
@pytest.mark.parametrize("kernel", ["k_x_c2c_v<16,1,1>", "k_x_c2c_v<16,6,1>", "k_x_c2c_v<24,6,-1>",
                                    "k_x_c2c_v<48,3,-1>", "k_x_c2c_v<192,6,1>", "k_x_c2c_v<320,2,1>",
                                    "k_x_c2c_v<512,3,-1>", "k_x_r2c<48,3>", "k_x_r2c<128,2>"])
def test_first_loads_are_issued_together(kernel, tmp_path):
    name, args = kernel[:-1].split("<")
    mangled = "_ZN3lf2%d%sI%sEEvNS_5XArgsE" % (len(name), name, "".join(
        "Li%sE" % a.replace("-", "n") for a in args.split(",")))
    assert _kernel_waits(mangled, tmp_path) == 0


# strided passes over the longest lines, backward, narrow and wide; over 512 points
@pytest.mark.parametrize("mangled", [
    "_ZN3lf29k_stridedILi1024ELi1ELb0ELb0ELi0EEEvNS_5SArgsE",
    "_ZN3lf29k_stridedILi1024ELi1ELb0ELb1ELi0EEEvNS_5SArgsE",
    "_ZN3lf29k_stridedILi2048ELi1ELb0ELb0ELi0EEEvNS_5SArgsE",
    "_ZN3lf211k_strided_wILi1024ELi1ELb1EEEvNS_5SArgsE",
    "_ZN3lf211k_strided_wILi2048ELi1ELb0EEEvNS_5SArgsE",
    "_ZN3lf29k_stridedILi512ELin1ELb0ELb0ELi0EEEvNS_5SArgsE"])
def test_first_column_loads_are_issued_together(mangled, tmp_path):
    assert _kernel_waits(mangled, tmp_path) == 0
