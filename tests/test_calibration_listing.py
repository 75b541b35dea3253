"""The calibration's fit as it is compiled: registers in memory only where that was measured to be worth an additional block."""
import os
import re
import subprocess

import pytest

from paper_2501_10054_amd import build as B


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("calibration") / "offline.s")
    subprocess.run([hipcc, *B.FLAGS, "--offload-device-only", "-S", os.path.join(B.CSRC, "offline.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_registers_of_the_fit(listing):
    """Blocks of 256 threads, five a CU: at most 96 registers, one more of them spilt.  Blocks of 512: two a CU with up to 128, none spilt."""
    seen = {}
    for part in re.split(r"\n  - \.agpr_count", listing[listing.index("amdhsa.kernels:"):])[1:]:
        m = re.search(r"calibrate_neuron_kernelI[tf]Li(\d+)ELi(\d+)E", re.search(r"\.name:\s+(\S+)", part)[1])
        if m:
            seen.setdefault((int(m[1]), int(m[2])), []).append([int(re.search(rf"\.{k}:\s+(\d+)", part)[1]) for k in ("vgpr_count", "vgpr_spill_count")])
    assert sorted(seen) == [(256, 4), (256, 16), (512, 16), (1024, 32)] and all(len(v) == 2 for v in seen.values())
    assert all(vgpr <= 96 and spilt <= 1 for vgpr, spilt in seen[256, 16])
    assert all(vgpr <= 128 and spilt == 0 for vgpr, spilt in seen[512, 16] + seen[256, 4])
