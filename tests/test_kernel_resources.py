"""What the compiler gave the kernels whose launches count on it, read from the code objects in
the built library (no GPU needed).  The workgroups of the resident tridiagonalisation wait for
each other, and the launches that may run at a time are limited to two workgroups per CU: every
instance has to fit 256 registers a thread (4 waves of 64 lanes, 512 registers a lane and SIMD),
without spilling, and half of the 160 KB of LDS."""
import os
import re
import shutil
import struct
import subprocess

import pytest

slrx = pytest.importorskip("paper_1704_04511_amd")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    blob = open(slrx.library_path(), "rb").read()
    at = blob.find(MAGIC)
    while at >= 0:
        n, pos = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + tlen]
            pos += 24 + tlen
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + len(MAGIC))


def kernels(tmp_path):
    readelf = shutil.which("llvm-readelf") or os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm/bin/llvm-readelf")
    if not os.path.exists(readelf):
        pytest.skip("llvm-readelf not installed")
    out = {}
    for i, co in enumerate(code_objects()):
        f = tmp_path / f"{i}.co"
        f.write_bytes(co)
        text = subprocess.run([readelf, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n\s+- \.agpr_count:", text)[1:]:
            get = lambda key: int(re.search(rf"\.{key}:\s+(\d+)", part).group(1))
            out[re.search(r"\.name:\s+(\S+)", part).group(1)] = {k: get(k) for k in (
                "vgpr_count", "vgpr_spill_count", "group_segment_fixed_size")}
    return out


def test_resident_tridiagonalisation_fits_two_workgroups_per_cu(tmp_path):
    found = {k: v for k, v in kernels(tmp_path).items() if re.search(r"\d+k_tri_resILi", k)}
    assert len(found) == 9, sorted(found)  # five sizes, of one problem and of batches (equal for the largest)
    for name, v in found.items():
        assert v["vgpr_count"] <= 256 and v["vgpr_spill_count"] == 0, (name, v)
        assert 2 * v["group_segment_fixed_size"] <= 160 * 1024, (name, v)
