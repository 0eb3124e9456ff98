"""The wait states behind the MFMAs that are written in inline assembly, read from the built library's own gfx950 code.

The compiler's hazard recogniser does not see such an MFMA: neither that a vector instruction ahead of it has just written one of
its operands (2 wait states), nor that its result takes 4 passes to arrive (7 wait states until another vector
instruction, a store or an LDS write reads or replaces it).  Where the compiler copies accumulators, and where it computes
operands, is its own choice and may change with any edit, so this looks at what it chose, in the order of the code.  No GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2604_19654_amd as fe

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
OPERAND_WAIT_STATES, RESULT_WAIT_STATES = 2, 7


def registers(operand):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", operand.strip())
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.fullmatch(r"([va])(\d+)", operand.strip())
    return {(m.group(1), int(m.group(2)))} if m else set()


def short_waits(lines):
    """[(line, kind)] of the instructions that come too early, and the number of MFMAs."""
    past, problems, mfmas = [], [], 0
    for at, line in enumerate(lines):
        text = line.split("//")[0].strip()
        if not text or text.endswith(":"):
            continue
        mnemonic, _, rest = text.partition(" ")
        operands = [registers(o) for o in re.split(r",\s*|\s(?=offen|offset|off\b)", rest)]
        is_mfma = mnemonic.startswith("v_mfma")
        mfmas += is_mfma
        touched = set().union(*(operands[1:] if is_mfma else operands))
        waited = 0
        for old, written, old_is_mfma, states in reversed(past):
            if waited >= RESULT_WAIT_STATES:
                break
            if written & touched:
                if is_mfma and not old_is_mfma and old.startswith("v_") and waited < OPERAND_WAIT_STATES:
                    problems.append((at, "operand"))
                if old_is_mfma and not is_mfma:
                    problems.append((at, "result"))
            waited += states
        past.append((mnemonic, operands[0] if mnemonic.startswith("v_") else set(), is_mfma, int(rest, 0) + 1 if mnemonic == "s_nop" else 1))
        del past[:-16]
    return problems, mfmas


def test_the_check_itself():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"
    copy, read = "v_accvgpr_mov_b32 a9, a3", "v_mov_b32_e32 v5, v20"
    assert short_waits([mfma, "s_nop 5", copy])[0] == [(2, "result")]
    assert short_waits([mfma, "s_nop 6", copy])[0] == []
    assert short_waits([mfma, copy])[0] == [(1, "result")]
    assert short_waits([read, "s_nop 0", mfma])[0] == [(2, "operand")]
    assert short_waits([read, "s_nop 1", mfma])[0] == []
    assert short_waits([mfma, mfma]) == ([], 2)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_wait_states_of_the_tall_tiles_mfmas(tmp_path):
    lib = tmp_path / "l.so"
    shutil.copy(fe.lib_path(), lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    kernels = mfmas = 0
    for name in os.listdir(tmp_path):
        if "gfx950" not in name:
            continue
        code = subprocess.run([OBJDUMP, "-d", str(tmp_path / name)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"^[0-9a-f]+ (?=<)", code, flags=re.M)[1:]:
            head, _, body = kernel.partition("\n")
            if "tall_gemm_kernel" not in head:
                continue
            problems, n = short_waits(body.splitlines())
            assert not problems, (head, problems[:5])
            kernels, mfmas = kernels + 1, mfmas + n
    assert kernels == 6 and mfmas > 1000
