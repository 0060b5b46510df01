"""Every kernel of the built library is short enough for plain branches: a branch
reaches 2^15 instruction words, 128 KiB.  With three inlined copies of a segment the
FP64 two-step kernels were 370 KiB long, needed long branches and 1164 spilled
scalars, and gave wrong results; with one copy they are under 100 KiB and right.  A
kernel that grows past the reach again is to be cut before it is trusted."""
import os
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2505_22256_amd", "liblbm.so")
BIN = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 entries of the uncompressed offload bundles in `data`."""
    pos = data.find(MAGIC)
    while pos >= 0:
        (n,), o = struct.unpack_from("<Q", data, pos + 24), pos + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, o)
            if size and b"gfx950" in data[o + 24:o + 24 + length]:
                yield data[pos + off:pos + off + size]
            o += 24 + length
        pos = data.find(MAGIC, pos + 24)


@pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("llvm-readelf", path=BIN), reason="no library or LLVM tools")
def test_kernels_need_no_long_branch(tmp_path):
    fat = tmp_path / "fat.bin"
    subprocess.run([os.path.join(BIN, "llvm-objcopy"), "--dump-section", ".hip_fatbin=%s" % fat, LIB, str(tmp_path / "x.so")],
                   check=True)
    sizes = {}
    for k, obj in enumerate(_code_objects(fat.read_bytes())):
        elf = tmp_path / ("co%d.elf" % k)
        elf.write_bytes(obj)
        out = subprocess.run([os.path.join(BIN, "llvm-readelf"), "-sW", str(elf)], check=True, capture_output=True, text=True)
        for line in out.stdout.splitlines():
            f = line.split()
            if len(f) == 8 and f[3] == "FUNC":
                sizes[f[7]] = int(f[2], 0)
    assert len(sizes) > 300
    assert {n: s for n, s in sizes.items() if s > 4 * 2 ** 15 - 4096} == {}
