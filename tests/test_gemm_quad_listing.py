"""The products with four wavefronts keep their accumulators in the other half of the register file and place m0 and
the load that uses it in different gaps between MFMAs, all in inline assembly: their listing is read here for what
test_gemm_listing reads the other kernels' for - waits behind and before the MFMAs, m0, spills."""
import re

import pytest

from test_gemm_listing import AFTER_MFMA, BEFORE_MFMA, _kernels, _walk, listings  # noqa: F401


def _registers(text):
    regs = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo, hi = (int(m[2]), int(m[3])) if m[2] else (int(m[4]), int(m[4]))
        regs.update((m[1], r) for r in range(lo, hi + 1))
    return regs


@pytest.mark.parametrize("packed", [False, True])
def test_results_of_matrix_instructions_are_waited_for(listings, packed):  # noqa: F811
    kernels = _kernels(listings[packed], "gemm_quad_kernel")
    assert len(kernels) == 30                       # 5 tiles x (4 epilogues, two of them for ragged rows too)
    for name, (code, labels) in kernels.items():
        operands = [[_registers(p) for p in re.split(r",\s*", rest)] if rest else [] for _, rest in code]
        every = [set().union(*o) if o else set() for o in operands]
        assert any(op.startswith("v_mfma") for op, _ in code), name
        for i, (op, rest) in enumerate(code):
            if op.startswith("v_mfma"):
                result = operands[i][0]
                for k in _walk(code, labels, i, AFTER_MFMA):
                    again = (code[k][0].startswith("v_mfma") and operands[k][0] == result == operands[k][3] and
                             not (operands[k][1] | operands[k][2]) & result)
                    assert again or not every[k] & result, (name, op, rest, code[k])
            elif op.startswith("v_") and operands[i] and operands[i][0]:
                for k in _walk(code, labels, i, BEFORE_MFMA):
                    if code[k][0].startswith("v_mfma"):
                        assert not operands[i][0] & set().union(*operands[k][1:4]), (name, op, rest, code[k])


def test_m0_belongs_to_the_loads_to_lds(listings):  # noqa: F811
    """Every load to LDS finds the m0 written for it, at least one instruction before, and nothing else uses m0."""
    for name, (code, _) in _kernels(listings[False], "gemm_quad_kernel").items():
        written = None
        for i, (op, rest) in enumerate(code):
            if re.search(r"\bm0\b", rest):
                assert op == "s_add_u32" and rest.startswith("m0, s") and written is None, (name, op, rest)
                written = i
            elif op.startswith("buffer_load") and "lds" in rest:
                # (the first load of a loop's body is the second half's last one, or the m0 before the loop is its)
                assert written is not None and i - written >= 2, (name, op, rest)
                written = None


def test_nothing_spills(listings):  # noqa: F811
    seen = 0
    for text in listings.values():
        for part in re.split(r"\n  - \.agpr_count", text[text.index("amdhsa.kernels:"):])[1:]:
            name = re.search(r"\.name:\s+(\S+)", part)[1]
            if "gemm_quad_kernel" in name:
                seen += 1
                assert int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part)[1]) == 0, name
                assert int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", part)[1]) == 0, name
    assert seen == 60
