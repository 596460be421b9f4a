"""Registers of the built library's iteration kernels (the compiler's own record in the code objects
built here).

* Multi-step kernel, FP64: at most 30 registers kept in memory, what it held before its
  factorisations were called out of line; beside those calls the inlined iteration held 59 to 62,
  some of them read in every iteration, and a small chain's steps took 3% longer.
* Per-scene kernel of problems with couplings of three and four members: at most 128 registers in
  FP32 and 168 in FP64 (four and three waves per SIMD, as many as without the descriptors of these
  couplings in LDS); with fewer resident scenes batches of 2,000 took up to 14% longer.
"""
import os
import re
import shutil
import subprocess

import pytest

BIN = "/opt/rocm/llvm/bin"


def _records(tmp_path, what):
    from paper_2302_14344_amd import build
    if not (os.path.exists(build.LIB) and os.path.exists(f"{BIN}/llvm-objdump") and os.path.exists(f"{BIN}/llvm-readelf")):
        pytest.skip("needs the built library and ROCm's binary tools")
    lib = tmp_path / "lib.so"
    shutil.copy(build.LIB, lib)
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in tmp_path.glob("lib.so.*gfx950"):
        r = subprocess.run([f"{BIN}/llvm-readelf", "--notes", str(f)], capture_output=True, text=True)
        for name, n in re.findall(r"\.name:\s+(\S+)\n(?:(?!\.name:).)*?\." + what + r":\s+(\d+)", r.stdout, re.S):
            out[name] = int(n)
    return out


def test_multi_step_kernels_in_fp64(tmp_path):
    found = {k: v for k, v in _records(tmp_path, "vgpr_spill_count").items() if "steps_kernelIdd" in k}
    assert len(found) == 3  # one and two lanes per row, split rows
    assert max(found.values()) <= 30, found


def test_couplings_of_more_than_two_members(tmp_path):
    found = _records(tmp_path, "vgpr_count")
    for t, most in (("f", 128), ("d", 168)):
        for lanes in (1, 2):
            n = [v for k, v in found.items() if f"loop_kernelI{t}Li1ELi{lanes}ELb1E" in k]
            assert len(n) == 1 and n[0] <= most, (t, lanes, n)
