"""Which calls of up to 64 tokens stream their weights, from the kernels that the host code launches (host_runtime.py): on either side of
the lines that the measurements beside the rules (stream.hip) draw."""
import re

import pytest

from host_runtime import hip, host  # noqa: F401
from paper_2501_10054_amd import tardis as T
from test_gpu_stream import STREAMS


def kernels(names):
    """matrix products of a call in their order: stream_kernel with its constants, or the other kernels' epilogue"""
    out = []
    for name in names:
        m = re.search(r"stream_kernelILi(\d)ELi(\d)ELi(\d)E", name)
        if m:
            out.append(f"{('part', 'repair')[int(m[1])]} {16 * int(m[2])} x {16 * int(m[3])}")
        m = re.search(r"gemm_(?:quad|tile)_kernelILi(\d)E", name)
        if m:
            out.append(("store", "part", "hidden", "repair")[int(m[1])])
    return out


def call(hip, d, h, n, dense=False, **fold):  # noqa: F811
    st, L = hip.fold(d=d, h=h, max_batch=max(n, 64), **fold)
    assert st == T.OK
    hip.launches()
    assert (hip.lib.tardis_dense_forward if dense else hip.lib.tardis_ffn_forward_batched)(L, 1 << 38, n, 1 << 37, None) == T.OK
    got = kernels(hip.launches())
    hip.lib.tardis_destroy(L)
    return got


UP = [(512, 2048, 20, "repair"), (896, 4096, 32, "repair"), (1024, 4096, 32, "repair 32 x 32"), (1024, 4096, 33, "repair"), (1920, 4096, 33, "repair"),
      (2048, 4096, 33, "repair 64 x 32"), (1024, 8192, 20, "repair 32 x 32"), (1024, 8200, 20, "repair 32 x 64"), (1024, 16384, 20, "repair 32 x 64"),
      (4096, 16384, 64, "repair 64 x 64"), (4096, 16392, 64, "repair"), (4096, 20480, 20, "repair"), (4096, 32768, 32, "repair 32 x 64"), (4096, 32768, 33, "repair"),
      (2048, 32768, 20, "repair"), (4096, 40960, 20, "repair"), (6144, 8192, 64, "repair 64 x 32"), (6272, 8192, 64, "repair"), (8192, 16384, 64, "repair 64 x 64")]


@pytest.mark.parametrize("d,h,n,want", UP)
def test_up_products(hip, d, h, n, want):  # noqa: F811
    assert call(hip, d, h, n)[0] == want


def test_prompts_do_not_stream(hip):  # noqa: F811
    assert call(hip, 4096, 16384, 65)[0] == "repair" and call(hip, 4096, 16384, 64, bits=4)[0] == "repair"


# (d, h, tokens, folded: kernels of the output, dense: the same)
OUTPUT = [(4096, 3200, 20, ["part", "part"], ["part"]), (4096, 3328, 20, ["part 32 x 64", "part"], ["part"]), (4096, 3328, 33, ["part", "part"], ["part"]),
          (4096, 8192, 32, ["part 32 x 64"], ["part 32 x 64"]), (4096, 8192, 33, ["part 64 x 64"], ["part"]), (4096, 8320, 40, ["part 64 x 64", "part"], ["part"]),
          (4096, 16384, 64, ["part 64 x 64"], ["part 64 x 64"]), (4096, 16392, 20, ["part", "part"], ["part"]), (4096, 16384, 65, ["part"], ["part"]),
          (2048, 14720, 20, ["part 32 x 64", "part 32 x 64"], ["part 32 x 64"]), (4096, 12416, 40, ["part 64 x 64", "part 64 x 64"], ["part 64 x 64"]),
          (2048, 24576, 64, ["part 64 x 64"], ["part 64 x 64"]), (1024, 28672, 20, ["part 32 x 32"], ["part"]), (1024, 30720, 32, ["part 32 x 32"], ["part 32 x 32"]),
          (1024, 65536, 33, ["part"], ["part"]), (3072, 12288, 32, ["part 32 x 64"], ["part 32 x 64"]), (3072, 24576, 32, ["part"], ["part 32 x 64"]),
          (3072, 16384, 33, ["part"], ["part"]), (2560, 10240, 20, ["part"], ["part"]), (5120, 20480, 20, ["part"], ["part"]), (8192, 8192, 20, ["part"], ["part"])]


@pytest.mark.parametrize("d,h,n,folded,dense", OUTPUT)
def test_output_products(hip, d, h, n, folded, dense):  # noqa: F811
    assert call(hip, d, h, n)[1:] == folded and call(hip, d, h, n, dense=True)[1:] == dense


@pytest.mark.parametrize("size", STREAMS)
def test_kernels_of_the_gpu_tests(hip, size):  # noqa: F811
    d, h, n = size
    assert call(hip, d, h, n) == list(STREAMS[size][:-1]) and call(hip, d, h, n, dense=True) == ["hidden", STREAMS[size][-1]]


def test_the_gpu_tests_reach_every_stream():
    seen = {k for kernels_of in STREAMS.values() for k in kernels_of if " x " in k}
    assert seen == {f"repair {m} x {n}" for m in (32, 64) for n in (32, 64)} | {"part 32 x 32", "part 32 x 64", "part 64 x 64"}
