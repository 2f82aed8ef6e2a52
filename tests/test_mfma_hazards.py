"""The bf16 kernels' multiplications are inline assembly, so the compiler does not keep the distances that the hardware
wants around them.  This reads the built library's code (the AMD assembly of this repository's own kernels) and looks for
    a vector instruction's result read by an MFMA less than 2 wait states later,
    an MFMA's result read or overwritten by anything but the next MFMA's accumulation less than 8 wait states later
(4-pass MFMA on gfx950).  Code is read in the order it lies in, branches included.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_19362_amd import oapl

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VALU_TO_MFMA, MFMA_TO_ANY = 2, 8


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$", operand)
    if m:
        return frozenset(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v(\d+)$", operand)
    return frozenset([int(m.group(1))]) if m else frozenset()


def hazards(listing):
    found, recent, now, multiplications = [], [], 0, 0
    for line in listing:
        text = line.split("//")[0].strip()
        if text.startswith("<"):
            recent = []
        m = re.match(r"([a-z]\w+)\s*(.*)$", text)
        if not m:
            continue
        op, rest = m.groups()
        operands = [_registers(x.strip().split(" ")[0]) for x in rest.split(",")]
        recent = [r for r in recent if now - r[2] < 16]
        if op.startswith("v_mfma"):
            multiplications += 1
            dst, a, b, c = operands[:4]
            for kind, regs, at in recent:
                if kind == "valu" and now - at < VALU_TO_MFMA and regs & (a | b | c):
                    found.append(text)
                if kind == "mfma" and now - at < MFMA_TO_ANY and (regs & (a | b) or (regs & c and regs != c)):
                    found.append(text)
            recent.append(("mfma", dst, now + 1))
        elif op.startswith(("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")):
            touched = frozenset().union(*operands)
            if any(kind == "mfma" and now - at < MFMA_TO_ANY and regs & touched for kind, regs, at in recent):
                found.append(text)
            if op.startswith("v_"):
                written = operands[0] | (operands[1] if "swap" in op and len(operands) > 1 else frozenset())
                recent.append(("valu", written, now + 1))
        now += int(rest.split()[0], 0) + 1 if op == "s_nop" else 1
    return found, multiplications


@pytest.mark.parametrize("listing, bad", [
    (["v_mov_b32_e32 v1, v9", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]"], 1),
    (["v_mov_b32_e32 v1, v9", "s_nop 1", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_nop 6", "v_mov_b32_e32 v9, v23"], 1),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_nop 7", "global_store_dwordx4 v[8:9], v[20:23], off"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]",
      "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[12:15], v[20:23]"], 0),
])
def test_the_reader_sees_hazards(listing, bad):
    assert len(hazards(listing)[0]) == bad


def test_no_hazards_in_the_built_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not found")
    lib = tmp_path / "lib.so"
    shutil.copy(oapl.lib_path(), lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(code) == 1
    out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", code[0]], cwd=tmp_path, check=True,
                         stdout=subprocess.PIPE, text=True).stdout
    found, multiplications = hazards(out.splitlines())
    assert multiplications > 1000
    assert not found, found[:10]
