"""The transfers global memory -> LDS of the streaming GEMMs as the library holds them (no GPU needed).

The compiler does not look for hazards inside asm statements: a memory instruction may read a scalar register that a vector instruction
wrote (v_readlane brings back a spilled one) only five wait states later, and m0 has to be written two instructions before the
transfer.  Both hold wherever the transfer's base is a scalar copy made right behind the write of m0."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def test_every_transfer_takes_its_base_from_a_scalar_copy(tmp_path):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    lib = shutil.copy(metis.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    transfers = {}
    for image in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(image)], check=True, capture_output=True, text=True).stdout
        lines = [re.sub(r"\s*//.*", "", line).strip() for line in text.splitlines() if line.startswith("\t")]
        for i, line in enumerate(lines):
            m = re.match(r"global_load_lds_(\w+) v\d+, (s\[\d+:\d+\])", line)
            if m:
                transfers[m.group(1)] = transfers.get(m.group(1), 0) + 1
                assert lines[i - 1].startswith(f"s_mov_b64 {m.group(2)}, s["), lines[i - 2:i + 1]
                assert lines[i - 2].startswith("s_add_u32 m0, s"), lines[i - 2:i + 1]
            else:
                assert "global_load_lds" not in line, line
    assert set(transfers) == {"dwordx4", "dword"}, transfers
