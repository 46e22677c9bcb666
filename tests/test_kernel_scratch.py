"""Registers and scratch memory of y transforms, from the metadata of the built
library's code objects. Persistent launches: a thread that walks many blocks keeps nothing
across them, so none of it spills but at the two longest lengths, whose 800
and 864 threads leave 128 registers each.
Default launches of 1024 points: two workgroups of 512 threads share a compute
unit, at 128 registers a thread."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2502_06296_amd import _native as N

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:/opt/rocm/lib/llvm/bin") or shutil.which("llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(tmp_path):
    """{mangled kernel: (bytes of scratch, registers) of a thread} of every code
    object."""
    data = open(N.LIB_PATH, "rb").read()
    out = {}
    for n, m in enumerate(re.finditer(MAGIC, data)):
        at = m.start()
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        if not 0 < count < 16:
            continue
        for _ in range(count):
            off, size, ln = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + ln]
            pos += 24 + ln
            if b"gfx950" not in name:
                continue
            obj = tmp_path / f"{n}.co"
            obj.write_bytes(data[at + off:at + off + size])
            text = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            for kernel in text.split("  - .agpr_count:")[1:]:
                sym = re.search(r"\.name:\s+(\S+)", kernel)
                priv = re.search(r"\.private_segment_fixed_size:\s*(\d+)", kernel)
                regs = re.search(r"\.vgpr_count:\s*(\d+)", kernel)
                out[sym[1]] = int(priv[1]), int(regs[1])
    return out


@pytest.mark.skipif(READELF is None, reason="needs llvm-readelf")
def test_persistent_y_transforms_keep_nothing_in_scratch(tmp_path):
    scratch = {k: v for k, (v, _) in _kernels(tmp_path).items() if "k_yr_persist" in k or "k_y_persist" in k}
    assert len(scratch) >= 50
    for k, v in scratch.items():
        length = int(re.search(r"persistI[fd]Li(\d+)E", k)[1])
        assert v == 0 if length < 3200 else v <= 128, (k, v)


@pytest.mark.skipif(READELF is None, reason="needs llvm-readelf")
def test_1024_point_y_workgroups_share_a_compute_unit(tmp_path):
    regs = {k: v for k, (_, v) in _kernels(tmp_path).items() if re.search(r"k_yrI[fd]Li1024ELi8ELb[01]ELi0ELb0E", k)}
    assert len(regs) == 4
    for k, v in regs.items():
        assert v <= 128, (k, v)
