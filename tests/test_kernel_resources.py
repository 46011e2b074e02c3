"""Vector registers that the compiler spills to memory in the stage and OE kernels of the
built library (its code objects' metadata).  Orders 3 to 5 run two waves per SIMD in 256
registers and are written to fit: a spilled register in the second half of a row waits for
the row prefetch.  The limiter's point test, which few rows take, may spill within itself.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_26194_amd", "libfam.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
EM_AMDGPU = 224

# (kernel, k, limiter) -> spilled registers of the Euler instantiation; any other: none
POINT_TEST = {("stage2d_kernel", 5, True): 2, ("stage2d_list_kernel", 5, True): 2,
              ("stage2d_batched_kernel", 4, True): 10, ("stage2d_batched_kernel", 5, True): 14}
# k = 6 runs one wave per SIMD and is full; so many at most
ORDER6 = 22


def _spills(tmp_path):
    """{mangled kernel name: spilled vector registers}"""
    blob = open(LIB, "rb").read()
    out, at = {}, blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            co = tmp_path / "code_object"
            co.write_bytes(blob[at:])
            notes = subprocess.run([READELF, "--notes", str(co)], capture_output=True, text=True, check=True).stdout
            names = re.findall(r"^    \.name:\s+(\S+)", notes, re.M)
            counts = re.findall(r"^    \.vgpr_spill_count:\s+(\d+)", notes, re.M)
            assert len(names) == len(counts)
            out.update(zip(names, map(int, counts)))
        at = blob.find(b"\x7fELF", at + 4)
    return out


def test_stage_and_oe_kernels_spill_no_more_than_stated(tmp_path):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    seen = 0
    for name, spilled in _spills(tmp_path).items():
        m = re.search(r"\d+(stage2d_kernel|stage2d_list_kernel|stage2d_batched_kernel|oe2d_kernel|oe2d_batched_kernel)"
                      r"ILi(\d)ENS_\d+(\w+?)(?:ILi2EE)?E((?:L[bi]\dE)*)", name)
        if not m:
            continue
        seen += 1
        kernel, k, system, flags = m.group(1), int(m.group(2)), m.group(3), re.findall(r"L[bi](\d)E", m.group(4))
        limiter = kernel == "stage2d_list_kernel" or (kernel.startswith("stage2d") and flags[0] == "1")
        if k == 6 and kernel.startswith("stage2d"):
            most = ORDER6 if system.startswith("Euler") else 0
        else:
            most = POINT_TEST.get((kernel, k, limiter), 0) if system.startswith("Euler") else 0
        assert spilled <= most, (kernel, k, system, flags, spilled)
    assert seen >= 80   # four orders, three systems, one mesh and batches, with and without the limiter
