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


def _instructions(text):
    """(address, operation, operands) of every instruction, in order"""
    for line in text.splitlines():
        m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m:
            yield int(m.group(3), 16), m.group(1), [re.split(r"\s", x.strip())[0] for x in m.group(2).split(",")]


def _program(text):
    """the instructions, and for every address the branches that go there"""
    code, jumps = list(_instructions(text)), {}
    for i, (at, op, operands) in enumerate(code):
        if op.startswith(("s_branch", "s_cbranch")):
            words = int(operands[0])
            jumps.setdefault(at + 4 + 4 * (words - 65536 if words >= 32768 else words), []).append(i)
    return code, jumps


def _written_before(code, jumps, i, states):
    """registers that vector instructions write within so many wait states before instruction i, on any way there"""
    found = set()
    before = [i - 1] if i and not re.match("s_branch|s_endpgm|s_setpc", code[i - 1][1]) else []
    for j in before + jumps.get(code[i][0], []):
        _, op, operands = code[j]
        if op.startswith("v_") and not op.startswith(("v_cmp", "v_mfma")):
            found |= _registers(operands[0])
        left = states - (int(operands[0]) + 1 if op == "s_nop" else 1)
        if left > 0:
            found |= _written_before(code, jumps, j, left)
    return found


def test_operands_are_not_written_just_before(tmp_path):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    lib = shutil.copy(metis.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    seen = {"v_fmac_f64_dpp": 0, "v_mfma_scale_f32_32x32x64_f8f6f4": 0}
    for image in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(image)], check=True, capture_output=True, text=True).stdout
        code, jumps = _program(text)
        assert set(jumps) <= {at for at, _, _ in code}
        for i, (at, op, operands) in enumerate(code):
            if op in seen:
                seen[op] += 1
                sources = operands[1:2] if op == "v_fmac_f64_dpp" else operands[1:3] + operands[4:6]
                written = _written_before(code, jumps, i, 2)
                for source in sources:
                    assert not _registers(source) & written, (hex(at), op, operands)
    assert all(n > 0 for n in seen.values()), seen


def test_the_look_back_follows_branches():
    # v[4:5] is written at a loop's end, one wait state (the branch) before the instruction at its head
    listing = ["v_mov_b32_e32 v9, v8", "s_nop 1", "v_fmac_f64_dpp v[0:1], v[4:5], v[2:3] row_newbcast:0", "v_add_f64 v[6:7], v[0:1], 1.0",
               "v_add_f64 v[4:5], v[0:1], 1.0", "s_cbranch_scc1 65532"]
    code, jumps = _program("\n".join(f"\t{line} // {4 * i:012X}: 00000000" for i, line in enumerate(listing)))
    assert jumps == {8: [5]}
    assert _written_before(code, jumps, 2, 2) == {4, 5} and _written_before(code, jumps, 2, 3) == {4, 5, 6, 7, 9}
