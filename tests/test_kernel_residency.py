"""Waves per SIMD of the march kernels, from the register counts in the built
library (the metadata of its gfx950 code objects): not fewer than the launch
models count on (launch_us in kern_march2d.hip and kern_twophase.hip,
launch3_us in kern_march3d.hip, march_us in kern_batch.hip)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2012_03525_amd import acm

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

# kernel, template arguments -> waves per SIMD the models count on
MARCH2D = {  # T, nodes per lane, steps, walled x, axisymmetric
    **{("f", 1, 1, w, a): 7 for w in (0, 1) for a in (0, 1)},
    **{("f", 1, 2, w, a): 4 if w and a else 5 for w in (0, 1) for a in (0, 1)},
    **{("f", 1, 3, w, a): 3 for w in (0, 1) for a in (0, 1)},
    **{("f", 2, 1, w, a): 4 for w in (0, 1) for a in (0, 1)},
    **{("f", 2, 2, w, a): 2 if w else 3 for w in (0, 1) for a in (0, 1)},
    **{("d", 1, 1, w, a): 3 for w in (0, 1) for a in (0, 1)},
    **{("d", 1, 2, w, a): 2 for w in (0, 1) for a in (0, 1)},
}


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """kernel name -> VGPRs"""
    if READELF is None:
        pytest.skip("no llvm-readelf")
    lib = open(acm.LIB_PATH, "rb").read()
    out, at = {}, lib.find(MAGIC)
    tmp = tmp_path_factory.mktemp("code")
    while at >= 0:
        n, = struct.unpack_from("<Q", lib, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, p)
            name = lib[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" not in name or size == 0:
                continue
            f = os.path.join(str(tmp), f"{at:x}.co")
            open(f, "wb").write(lib[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", f], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n\s+- \.", notes)[1:]:
                nm, vg = re.search(r"\.name:\s+(\S+)", k), re.search(r"\.vgpr_count:\s+(\d+)", k)
                if nm and vg:
                    out[nm.group(1)] = int(vg.group(1))
        at = lib.find(MAGIC, at + 1)
    assert out
    return out


def waves(vgprs):
    return min(8, 512 // (-(-vgprs // 8) * 8))


def test_march2d(registers):
    seen = set()
    for name, v in registers.items():
        m = re.search(r"march2d_kernelI([fd])Li(\d)ELi(\d)ELb([01])ELb([01])ELb([01])", name)
        if m:
            key = (m[1], int(m[2]), int(m[3]), int(m[4]), int(m[6]))
            seen.add(key)
            assert waves(v) >= MARCH2D[key], (name, v)
    assert seen == set(MARCH2D)


def test_batch_march3d_and_two_phase(registers):
    want = {r"batch_march_kernelIfLi2E": 5, r"batch_march_kernelIdLi2E": 2, r"march3d_kernelIfLi1ELi2E": 3,
            r"march3d_kernelIfLi1ELi4E": 2, r"twophase_march_kernelIfLi1E": 4, r"twophase_march_kernelIfLi2E": 2,
            r"twophase_march_kernelId": 2, r"stage1_march_kernel": 3, r"flow_stage2_march_kernel": 3}
    for pattern, w in want.items():
        found = [(n, v) for n, v in registers.items() if pattern in n]
        assert found, pattern
        for n, v in found:
            assert waves(v) >= w, (n, v)
