"""Registers that the built library's multi-step kernels keep in memory (the compiler's own record
in the code objects built here).  FP64: at most 30, what the kernel held before its
factorisations were called out of line; beside those calls the inlined iteration held 59 to 62,
some of them read in every iteration, and a small chain's steps took 3% longer.
"""
import os
import re
import shutil
import subprocess

import pytest

BIN = "/opt/rocm/llvm/bin"


def _spills(tmp_path):
    from paper_2302_14344_amd import build
    if not (os.path.exists(build.LIB) and os.path.exists(f"{BIN}/llvm-objdump") and os.path.exists(f"{BIN}/llvm-readelf")):
        pytest.skip("needs the built library and ROCm's binary tools")
    lib = tmp_path / "lib.so"
    shutil.copy(build.LIB, lib)
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in tmp_path.glob("lib.so.*gfx950"):
        r = subprocess.run([f"{BIN}/llvm-readelf", "--notes", str(f)], capture_output=True, text=True)
        for name, n in re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", r.stdout, re.S):
            out[name] = int(n)
    return out


def test_multi_step_kernels_in_fp64(tmp_path):
    found = {k: v for k, v in _spills(tmp_path).items() if "steps_kernelIdd" in k}
    assert len(found) == 3  # one and two lanes per row, split rows
    assert max(found.values()) <= 30, found
