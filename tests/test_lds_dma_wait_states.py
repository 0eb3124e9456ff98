"""The wait states of the LDS-DMA loads, read from the built library's own gfx950 code.

The loads are written in inline assembly, where the compiler's hazard recogniser adds nothing, so the wait states that
the hardware does not supply have to be in the code: one between a scalar write of M0 and the load that takes its LDS
address from it, and five between a vector instruction that writes a scalar register (v_readfirstlane and its like)
and a memory instruction that reads that register as its address or descriptor.  Which unit the compiler computes an
address on is its own choice and may change with any edit, so this looks at what it chose, on every way that leads to
each load.  No GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2604_19654_amd as fe

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"

ADDRESS_WAIT_STATES = 5
M0_WAIT_STATES = 1


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


def parse(line):
    """(mnemonic, operands) of one line of disassembly; a label is ("", [label])."""
    text = line.split("//")[0].strip()
    label = re.fullmatch(r"(?:[0-9a-f]+ )?<(L\d+)>:", text)
    if label:
        return "", [label.group(1)]
    mnemonic, _, rest = text.partition(" ")
    return mnemonic, [p.strip() for p in re.split(r",|\s(?=offen|offset|lds|off\b)", rest) if p.strip()]


def is_lds_dma(mnemonic, operands):
    return (mnemonic.startswith("buffer_load") and "lds" in operands) or mnemonic.startswith("global_load_lds")


def short_waits(lines):
    """[(line, kind)] of the LDS-DMA loads with a way to them that lacks wait states, and the number of loads."""
    code = [parse(l) for l in lines]
    jumps = {}
    for i, (mnemonic, operands) in enumerate(code):
        if mnemonic.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(operands[0], []).append(i)

    def before(i):
        """Lines that control can come from to line i."""
        way = [] if i == 0 or code[i - 1][0] in ("s_branch", "s_endpgm", "s_setpc_b64") else [i - 1]
        return way + (jumps.get(code[i][1][0], []) if code[i][0] == "" else [])

    problems, loads = [], 0
    for at, (mnemonic, operands) in enumerate(code):
        if not is_lds_dma(mnemonic, operands):
            continue
        loads += 1
        reads = set().union(*(scalar_registers(o) for o in operands))
        todo, seen, kinds = [(p, 0) for p in before(at)], set(), set()
        while todo:
            i, waited = todo.pop()
            if (i, waited) in seen or waited >= ADDRESS_WAIT_STATES:
                continue
            seen.add((i, waited))
            m, ops = code[i]
            # (a vector instruction's scalar results are its first or, as carry, its second operand)
            if m.startswith("v_") and any(scalar_registers(o) & reads for o in ops[:2]):
                kinds.add("address")
            if m.startswith("s_") and ops[:1] == ["m0"] and waited < M0_WAIT_STATES:
                kinds.add("m0")
            waited += 0 if m == "" else int(ops[0], 0) + 1 if m == "s_nop" else 1
            todo += [(p, waited) for p in before(i)]
        problems += [(at, kind) for kind in sorted(kinds)]
    return problems, loads


def test_the_check_itself_on_known_sequences():
    def load(*lines):
        return short_waits([*lines, "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"])

    pad = ["s_add_u32 s20, s20, 1"] * 5
    assert load(*pad) == ([], 1)
    assert load("v_readfirstlane_b32 s6, v2", "s_mov_b32 m0, s30", "s_nop 0") == ([(3, "address")], 1)
    assert load("v_readfirstlane_b32 s6, v2", "s_mov_b32 m0, s30", "s_nop 3") == ([], 1)
    assert load("v_readfirstlane_b32 s8, v2", *pad[1:]) == ([], 1)
    assert load(*pad, "s_mov_b32 m0, s30") == ([(6, "m0")], 1)
    # the scalar base of a global load, and a carry-out
    assert short_waits(["v_add_co_u32_e64 v3, s[2:3], v3, v4", *pad[1:4], "s_nop 1",
                        "global_load_lds_dwordx4 v1, s[2:3]"]) == ([], 1)
    assert short_waits(["v_add_co_u32_e64 v3, s[2:3], v3, v4", *pad[1:4],
                        "global_load_lds_dwordx4 v1, s[2:3]"]) == ([(4, "address")], 1)
    # ways through branches: falling through one, and around a loop
    assert load("v_readfirstlane_b32 s6, v2", "s_cbranch_scc1 L0", "s_nop 2") == ([(3, "address")], 1)
    assert load("v_readfirstlane_b32 s6, v2", "s_branch L0", "s_nop 2") == ([], 1)
    loop = [*pad, "<L0>:", "s_nop 1", "global_load_lds_dwordx4 v1, s[2:3]", "v_readfirstlane_b32 s3, v2", "s_cbranch_scc1 L0"]
    assert short_waits(loop) == ([(7, "address")], 1)
    loop[6] = "s_nop 3"
    assert short_waits(loop) == ([], 1)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not found")
def test_every_lds_dma_load_has_its_wait_states(tmp_path):
    lib = shutil.copy(fe.lib_path(), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    total, bad = 0, {}
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", name], cwd=tmp_path, check=True,
                              capture_output=True, text=True).stdout
        # one section per kernel: "0000... <symbol>:" and its instructions
        for block in re.split(r"\n(?=[0-9a-f]+ <(?!L\d+>))", text):
            head, *lines = block.split("\n")
            problems, loads = short_waits([l for l in lines if l.strip()])
            total += loads
            if problems:
                bad[head] = [kind for _, kind in problems]
    assert total > 500, f"found {total} LDS-DMA loads: the disassembly was not understood"
    assert not bad, "\n".join(f"{len(v)} loads ({', '.join(sorted(set(v)))}) in {k}" for k, v in bad.items())
