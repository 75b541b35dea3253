"""The matrix-product kernels issue their MFMAs as inline assembly, so the compiler inserts none of the waits that
these instructions need.  The listing of gemm.hip is read here: behind every MFMA nothing may touch its result, and
before every MFMA no vector instruction may write its operands, within the wait states of the hardware - whatever
selection of instructions the compiler makes, so also without the switch that turns packed fp32 off (that listing is
only read, never run)."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2501_10054_amd import build as B

PACKED_OFF = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# wait states (an instruction is one, s_nop N is N + 1) behind an MFMA of up to 16 passes until another
# instruction than an MFMA that accumulates onto the same registers may read or write its result, and between a vector
# instruction and an MFMA that reads what it wrote
AFTER_MFMA, BEFORE_MFMA = 19, 2


def _listing(tmp, packed):
    src, out = os.path.join(B.CSRC, "gemm.hip"), os.path.join(tmp, f"gemm_{packed}.s")
    flags = [f for f in B.FLAGS]
    at = next(i for i in range(len(flags)) if flags[i:i + 4] == PACKED_OFF)
    if packed:
        del flags[at:at + 4]
    subprocess.run([B._hipcc(), *flags, "--offload-device-only", "-S", src, "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("no hipcc")
    tmp = str(tmp_path_factory.mktemp("listing"))
    with ThreadPoolExecutor(2) as ex:
        return dict(zip((False, True), ex.map(lambda p: _listing(tmp, p), (False, True))))


def _registers(text):
    regs = set()
    for m in re.finditer(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo, hi = (int(m[1]), int(m[2])) if m[1] else (int(m[3]), int(m[3]))
        regs.update(range(lo, hi + 1))
    return regs


def _kernels(text, kernel="gemm_tile_kernel"):
    """name -> list of (mnemonic, operands), label -> index"""
    out = {}
    for m in re.finditer(rf"^(_ZN?\S*{kernel}\S*):.*?\n(.*?)^\.Lfunc_end", text, re.S | re.M):
        code, labels = [], {}
        for line in m[2].splitlines():
            line = line.split(";")[0].strip()
            if re.fullmatch(r"\S+:", line):
                labels[line[:-1]] = len(code)
            elif line and not line.startswith("."):
                op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
                code.append((op.strip(), rest.strip()))
        out[m[1]] = (code, labels)
    return out


def _walk(code, labels, at, budget):
    """every instruction that can be issued within `budget` wait states behind number `at`"""
    seen, todo = {}, [(at + 1, 0)]
    while todo:
        i, spent = todo.pop()
        while i < len(code) and spent < budget and seen.get(i, budget) > spent:
            seen[i] = spent
            op, rest = code[i]
            if op == "s_endpgm":
                break
            spent += int(rest, 0) + 1 if op == "s_nop" else 1
            if op.startswith(("s_cbranch", "s_branch")):
                todo.append((labels[rest], spent))
                if op == "s_branch":
                    break
            i += 1
    return seen


def _faults(code, labels):
    found = []
    operands = {}
    for i, (op, rest) in enumerate(code):
        operands[i] = [_registers(p) for p in re.split(r",\s*", rest)] if rest else []
    every = {i: set().union(*o) if o else set() for i, o in operands.items()}
    for i, (op, rest) in enumerate(code):
        if op.startswith("v_mfma"):
            result = operands[i][0]
            for k in _walk(code, labels, i, AFTER_MFMA):
                if not every[k] & result:
                    continue
                same = (code[k][0].startswith("v_mfma") and operands[k][0] == result == operands[k][3] and
                        not (operands[k][1] | operands[k][2]) & result)
                if not same:
                    found.append(f"{op} {rest} -> {' '.join(code[k])}")
        elif op.startswith("v_") and operands[i] and operands[i][0]:
            for k in _walk(code, labels, i, BEFORE_MFMA):
                if code[k][0].startswith("v_mfma") and operands[i][0] & set().union(*operands[k][1:4]):
                    found.append(f"{op} {rest} -> {' '.join(code[k])}")
    return found


@pytest.mark.parametrize("packed", [False, True])
def test_results_of_matrix_instructions_are_waited_for(listings, packed):
    kernels = _kernels(listings[packed])
    assert len(kernels) >= 50
    bad = {}
    for name, (code, labels) in kernels.items():
        assert any(op.startswith("v_mfma") for op, _ in code), name
        assert not any("accvgpr" in op for op, _ in code), name
        found = _faults(code, labels)
        if found:
            bad[name] = (len(found), found[0])
    assert not bad, bad


def test_m0_belongs_to_the_loads_to_lds(listings):
    """m0 is written by the statement that loads to LDS and cannot be declared as overwritten: nothing else may use it."""
    for name, (code, _) in _kernels(listings[False]).items():
        for i, (op, rest) in enumerate(code):
            if re.search(r"\bm0\b", rest):
                assert op == "s_mov_b32" and rest.startswith("m0, s"), (name, op, rest)
                assert [code[i + 1][0], code[i + 2][0]] == ["s_nop", "buffer_load_dwordx4"] and "lds" in code[i + 2][1], name


def test_no_product_kernel_spills_vector_registers(listings):
    """A spill could store an accumulator that an MFMA is still writing, and costs trips to memory in the loop."""
    spills = {}
    for packed, text in listings.items():
        for part in re.split(r"\n  - \.agpr_count", text[text.index("amdhsa.kernels:"):])[1:]:
            name = re.search(r"\.name:\s+(\S+)", part)[1]
            if "gemm_tile_kernel" in name:
                spills[packed, name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part)[1])
    assert len(spills) >= 100
    assert not any(spills.values()), {n: c for n, c in spills.items() if c}
