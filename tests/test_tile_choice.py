"""Which tiles the matrix products of a call run on, from the kernels that the host code launches (host_runtime.py): the tests on the GPU
that mean certain tiles get those."""
import re

import pytest

from host_runtime import hip, host  # noqa: F401
from paper_2501_10054_amd import tardis as T
from test_gpu_quad_tiles import TILES

STORE, PART, HIDDEN, REPAIR = range(4)               # epilogues


def _products(names):
    """epilogue, tile of every product"""
    out = []
    for name in names:
        m = re.search(r"gemm_(quad|tile)_kernelILi(\d)ELb([01])E((?:Li\d+E)+)", name)
        if m:
            v = [int(x) for x in re.findall(r"Li(\d+)E", m[4])]
            rows, columns = (32 * v[0], 32 * v[1]) if m[1] == "quad" else (16 * v[1] * v[2], 16 * v[3] * (8 // v[1]))
            out.append((int(m[2]), f"{rows}x{columns}" + (" of eight" if m[1] == "tile" else "") + (" ragged" if m[3] == "1" else "")))
    return out


@pytest.mark.parametrize("size", TILES)
def test_tiles_of_the_gpu_tests(hip, size):  # noqa: F811
    d, h, n = size
    up, hidden, output, dense = TILES[size]
    st, L = hip.fold(d=d, h=h, max_batch=n)
    assert st == T.OK
    hip.launches()
    for call, want in ((hip.lib.tardis_ffn_forward_batched, [(REPAIR, up), (PART, output)]),
                       (hip.lib.tardis_dense_forward, [(HIDDEN, hidden), (PART, dense)])):
        assert call(L, 1 << 38, n, 1 << 37, None) == T.OK
        assert _products(hip.launches()) == want
    hip.lib.tardis_destroy(L)


def test_folds_of_the_gpu_tests(hip):  # noqa: F811
    """Large tiles with ragged rows, and a fold whose products are too small for the matrix cores (test_fold_rounds_in_the_second_product)."""
    for (d, h), tile in (((640, 8200), "128x128 ragged"), ((1024, 4104), "128x128 ragged"), ((130, 136), "128x128 ragged"),
                         ((257, 264), "128x128 ragged"), ((75, 130), None)):
        hip.launches()
        st, L = hip.fold(d=d, h=h)
        assert st == T.OK and _products(hip.launches()) == [(STORE, tile)] * 2 * (tile is not None)
        hip.lib.tardis_destroy(L)
