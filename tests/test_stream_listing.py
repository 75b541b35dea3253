"""The streaming kernels load to LDS with the same statement as the products (tiles.h), which writes m0 without being able to say so: their
listing is read for what test_gemm_listing reads the products' for.  (Their MFMAs are builtins, whose waits the compiler inserts.)"""
import os
import re
import subprocess

import pytest

from paper_2501_10054_amd import build as B
from test_gemm_listing import _kernels


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("stream") / "stream.s")
    subprocess.run([hipcc, *B.FLAGS, "--offload-device-only", "-S", os.path.join(B.CSRC, "stream.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_m0_belongs_to_the_loads_to_lds(listing):
    kernels = _kernels(listing, "stream_kernel")
    assert len(kernels) == 7
    for name, (code, _) in kernels.items():
        loads = 0
        for i, (op, rest) in enumerate(code):
            if re.search(r"\bm0\b", rest):
                assert op == "s_mov_b32" and rest.startswith("m0, s"), (name, op, rest)
                assert [code[i + 1][0], code[i + 2][0]] == ["s_nop", "buffer_load_dwordx4"] and "lds" in code[i + 2][1], name
                loads += 1
        assert loads and loads == sum(op.startswith("buffer_load") and "lds" in rest for op, rest in code), name


def test_nothing_spills(listing):
    seen = 0
    for part in re.split(r"\n  - \.agpr_count", listing[listing.index("amdhsa.kernels:"):])[1:]:
        if "stream_kernel" in re.search(r"\.name:\s+(\S+)", part)[1]:
            seen += 1
            assert all(int(re.search(rf"\.{k}:\s+(\d+)", part)[1]) == 0 for k in ("vgpr_spill_count", "private_segment_fixed_size"))
    assert seen == 7
