"""The beamform kernels keep their sums in registers: scratch memory per lane, from the
metadata of the code objects in the built library. A few dwords may be spilled outside
the gather loop (at most 64 bytes); sums that do not fit their registers take hundreds
of bytes and are read back at every gather. CPU only."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2311_00482_amd import build

READELF = os.path.join(os.path.dirname(os.path.realpath(shutil.which("hipcc") or
                                                        "/opt/rocm/bin/hipcc")),
                       "..", "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    if not (os.path.exists(build.LIB) and os.path.exists(READELF)):
        pytest.skip("no built library or no llvm-readelf")
    tmp = tmp_path_factory.mktemp("co") / "k.co"
    found = {}
    with open(build.LIB, "rb") as f:
        blob = f.read()
    for co in _code_objects(blob):
        tmp.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(tmp)], capture_output=True, text=True,
                               check=True).stdout
        for k in re.split(r"\n  - ", notes):
            name = re.search(r"\.name:\s+(\S*k_beamformI\S+)", k)
            if name:
                key = tuple(map(int, re.search(
                    r"ILi(\d+)ELb(\d)ELi(\d)ELi(\d)ELi(\d)E", name.group(1)).groups()))
                found[key] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1))
    return found


def test_sums_stay_in_registers(scratch):
    # angles, predicated, mode, lane groups, wavefronts per SIMD
    assert len({k[:4] for k in scratch}) == 4 * (3 * 32 + 2 * 17)  # groups x (RF + IQ modes)
    assert {k: v for k, v in scratch.items() if v > 64} == {}
