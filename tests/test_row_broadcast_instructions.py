"""Instructions written in asm whose operands the compiler does not watch, as the library holds them (no GPU needed).

A row broadcast (v_fmac_f64 with row_newbcast, the small factorizations) reads other lanes' registers: a vector instruction that wrote them has to be
two wait states away.  The MXFP4 matrix instruction reads codes and scale words: a vector instruction that wrote them has to be two
instructions away.  Nothing in an asm statement keeps the compiler from putting a copy in between."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _registers(operand):
    m = re.fullmatch(r"-?\|?v(?:\[(\d+):(\d+)\]|(\d+))\|?", operand)
    if not m:
        return set()
    lo = int(m.group(1) or m.group(3))
    return set(range(lo, int(m.group(2) or lo) + 1))


def test_operands_are_not_written_just_before(tmp_path):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    lib = shutil.copy(metis.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    seen = {"v_fmac_f64_dpp": 0, "v_mfma_scale_f32_32x32x64_f8f6f4": 0}
    for image in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(image)], check=True, capture_output=True, text=True).stdout
        recent = []                                    # registers written by the last wait states' vector instructions
        for line in text.splitlines():
            if not line.startswith("\t"):
                continue
            line = re.sub(r"\s*//.*", "", line).strip()
            op, _, rest = line.partition(" ")
            operands = [re.split(r"\s", x.strip())[0] for x in rest.split(",")]
            if op in seen:
                seen[op] += 1
                sources = operands[1:2] if op == "v_fmac_f64_dpp" else operands[1:3] + operands[4:6]
                for source in sources:
                    assert not _registers(source) & set().union(*recent[-2:]), line
            if op == "s_nop":
                recent += [set()] * (int(rest) + 1)
            else:
                recent.append(_registers(operands[0]) if op.startswith("v_") and not op.startswith(("v_cmp", "v_mfma")) else set())
            recent = recent[-4:]
    assert all(n > 0 for n in seen.values()), seen
