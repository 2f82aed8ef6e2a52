"""The bf16 kernels' multiplications are inline assembly, so the compiler does not keep the distances that the hardware
wants around them.  This reads the built library's code (the AMD assembly of this repository's own kernels) and looks for
    a vector instruction's result read by an MFMA less than 2 wait states later,
    an MFMA's result read or overwritten by anything but the next MFMA's accumulation less than 8 wait states later
(4-pass MFMA on gfx950), along every path that branches leave open.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_19362_amd import oapl

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VALU_TO_MFMA, MFMA_TO_ANY = 2, 8
VECTOR = ("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")


def _registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return frozenset((m.group(1), r) for r in range(int(m.group(2)), int(m.group(3)) + 1))
    m = re.match(r"([va])(\d+)$", operand)
    return frozenset([(m.group(1), int(m.group(2)))]) if m else frozenset()


def _functions(listing):
    """[(text, name, operands, wait states)] and {label: place} of every function."""
    code, labels = [], {}
    for line in listing:
        text = line.split("//")[0].strip()
        m = re.match(r"<(\w+)>:$", text)
        if m and not re.match(r"L\d+$", m.group(1)):
            yield code, labels
            code, labels = [], {}
        elif m:
            labels[m.group(1)] = len(code)
        else:
            m = re.match(r"([a-z]\w+)\s*(.*)$", text)
            if m:
                op, rest = m.groups()
                operands = [x.strip().split(" ")[0] for x in rest.split(",")]
                code.append((text, op, operands, int(operands[0], 0) + 1 if op == "s_nop" else 1))
    yield code, labels


def hazards(listing):
    found, multiplications = [], 0
    for code, labels in _functions(listing):
        regs = [[_registers(x) for x in operands] for _, _, operands, _ in code]

        def after(i, states):
            """Places that may be reached less than `states` wait states behind instruction i, on any path."""
            seen, todo = set(), [(i, 0)]
            while todo:
                at, passed = todo.pop()
                _, op, operands, _ = code[at]
                follow = [] if op in ("s_branch", "s_endpgm") else [at + 1]
                if op.startswith(("s_branch", "s_cbranch")):
                    follow.append(labels[operands[0]])
                for n in follow:
                    if n < len(code) and passed < states and (n, passed) not in seen:
                        seen.add((n, passed))
                        todo.append((n, passed + code[n][3]))
            return {n for n, _ in seen}

        for i, (_, op, _, _) in enumerate(code):
            if op.startswith("v_mfma"):
                multiplications += 1
                result = regs[i][0]
                for n in after(i, MFMA_TO_ANY):
                    if code[n][1].startswith("v_mfma"):
                        dst, a, b, c = regs[n][:4]
                        bad = result & (a | b) or (result & (c | dst) and not result == c == dst)
                    else:
                        bad = code[n][1].startswith(VECTOR) and result & frozenset().union(*regs[n])
                    if bad:
                        found.append(code[n][0])
            elif op.startswith("v_"):
                written = regs[i][0] | (regs[i][1] if "swap" in op and len(regs[i]) > 1 else frozenset())
                if not written:
                    continue
                for n in after(i, VALU_TO_MFMA):
                    if code[n][1].startswith("v_mfma") and written & frozenset().union(*regs[n][1:4]):
                        found.append(code[n][0])
    return found, multiplications


@pytest.mark.parametrize("listing, bad", [
    (["v_mov_b32_e32 v1, v9", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]"], 1),
    (["v_mov_b32_e32 v1, v9", "s_nop 1", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_nop 6", "v_mov_b32_e32 v9, v23"], 1),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_nop 7", "global_store_dwordx4 v[8:9], v[20:23], off"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]",
      "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[12:15], v[20:23]"], 0),
    # the top of a loop, reached from its end and from in front of it
    (["<L1>:", "v_add_f32_e32 v9, v23, v9", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_cbranch_scc0 L1",
      "s_endpgm"], 1),
    (["<L1>:", "v_add_f32_e32 v9, v23, v9", "v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_nop 6",
      "s_cbranch_scc0 L1", "s_endpgm"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_branch L2", "v_mov_b32_e32 v9, v23", "<L2>:", "s_endpgm"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[4:7], v[20:23]", "s_endpgm", "<other>:", "v_mov_b32_e32 v9, v23"], 0),
    # accumulation registers
    (["v_accvgpr_write_b32 a1, v9", "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"], 1),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "v_accvgpr_read_b32 v9, a3"], 1),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "v_mov_b32_e32 v3, v9"], 0),
])
def test_the_reader_sees_hazards(listing, bad):
    assert len(hazards(listing)[0]) == bad


def test_no_hazards_in_the_built_library(tmp_path):
    assert os.path.exists(OBJDUMP), "the distances cannot be checked without the compiler's llvm-objdump"
    lib = tmp_path / "lib.so"
    shutil.copy(oapl.lib_path(), lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(code) == 1
    out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", code[0]], cwd=tmp_path, check=True,
                         stdout=subprocess.PIPE, text=True).stdout
    found, multiplications = hazards(out.splitlines())
    assert multiplications > 1000
    assert not found, found[:10]
