"""Registers of the eigensolver's instances as the library holds them (no GPU needed).

The instances whose problems bring no second orthogonalisation pass (REPAIR = false) must not pay for its code: inlined into them as well, it
left 36 bytes of scratch a lane and slower sweeps."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin/"


def test_plain_sweeps_need_no_scratch(tmp_path):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not os.path.exists(LLVM + "llvm-readelf"):
        pytest.skip("library not built, or no reader of code objects")
    lib = shutil.copy(metis.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    scratch = {}
    for image in sorted(tmp_path.glob("lib.so.*gfx950")):
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(image)], check=True, capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S*k_jacobi_eigILi[1-6]ELi16ELb0\S*)\n.*?\.private_segment_fixed_size:\s*(\d+)", notes, re.S):
            scratch[name] = int(size)
    assert len(scratch) >= 6 and not any(scratch.values()), scratch
