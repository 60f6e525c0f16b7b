"""No kernel of the library reaches global memory by flat instructions (no GPU needed).

A flat instruction is one whose address the compiler could not place.  It counts as an LDS access too, so a wait for LDS and a counted wait
for the oldest of several loads both become waits for everything in flight."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def test_no_flat_instructions(tmp_path):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    lib = shutil.copy(metis.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    kernels, flat = 0, {}
    for image in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(image)], check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
                kernels += 1
            elif line.startswith("\tflat_"):
                flat[name] = flat.get(name, 0) + 1
    assert kernels > 0 and not flat, flat
