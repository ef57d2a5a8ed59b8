"""Registers of the built kernels: those that the solve loops launch per step keep
everything in registers (no spills to scratch memory).  Reads the metadata of the
library's own code objects; no GPU."""
import os
import re
import shutil
import struct
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2609_31347_amd", "libslbm.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 ELF images of the library (one bundle per source file)."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if name.endswith("gfx950") and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def test_solve_kernels_do_not_spill(tmp_path):
    readelf = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
    if readelf is None:
        pytest.skip("no llvm-readelf")
    with open(LIB, "rb") as f:
        blob = f.read()
    spills = {}
    for i, obj in enumerate(code_objects(blob)):
        path = os.path.join(tmp_path, f"{i}.co")
        with open(path, "wb") as f:
            f.write(obj)
        notes = subprocess.run([readelf, "--notes", path], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            spills[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1))
    watched = {n: s for n, s in spills.items()
               if re.search(r"k_sweep|k_primal|k_adjoint|k_tangent|k_residual|k_conv", n)}
    assert len(watched) >= 60
    assert {n: s for n, s in watched.items() if s} == {}
