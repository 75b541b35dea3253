"""Which codes a layer with a 4-bit sketch keeps, and which of its calls read them, from what the host code asks for and launches
(host_runtime.py)."""
import ctypes as C

import pytest

from host_runtime import hip, host  # noqa: F401
from paper_2501_10054_amd import tardis as T


def _products(hip, L, n):  # noqa: F811
    hip.launches()
    assert hip.lib.tardis_ffn_forward_batched(L, 1 << 38, n, 1 << 37, None) == T.OK
    return any("quantize_rows" in name for name in hip.launches())


@pytest.mark.parametrize("max_batch", [2, 3, 4, 5, 17])
def test_the_products_threshold_holds_for_packed_layers(hip, monkeypatch, max_batch):  # noqa: F811
    """TARDIS_PREFILL_MIN: calls with at least that many tokens are products, whatever codes a layer keeps otherwise."""
    monkeypatch.setenv("TARDIS_PREFILL_MIN", "2")
    st, L = hip.fold(d=2048, h=2048, max_batch=max_batch, bits=4)
    assert st == T.OK
    assert all(_products(hip, L, n) for n in range(2, max_batch + 1)) and not _products(hip, L, 1)
    hip.lib.tardis_destroy(L)


@pytest.mark.parametrize("d", [2048, 4096])
def test_one_byte_codes_of_packed_layers_can_be_left_out(hip, monkeypatch, d):  # noqa: F811
    """They triple the resident sketch.  TARDIS_PACKED_MAX: layers folded for at most that many tokens keep the packed codes alone,
    unless they can run as products."""
    h = 4096

    def memory(max_batch):
        st, L = hip.fold(d=d, h=h, max_batch=max_batch, bits=4)
        assert st == T.OK
        used = hip.lib.fake_used()
        hip.lib.tardis_destroy(L)
        assert hip.lib.tardis_release_memory() == T.OK
        return used

    default = {n: memory(n) for n in (4, 5, 16, 18)}
    monkeypatch.setenv("TARDIS_PACKED_MAX", "16")
    assert [default[n] - memory(n) for n in (4, 5, 16, 18)] == [0, d * h, d * h, 0]
    monkeypatch.setenv("TARDIS_PREFILL_MIN", "1000000")
    monkeypatch.setenv("TARDIS_PACKED_MAX", "1000000")
    assert (default[18] - memory(18)) // 4096 == d * h // 4096
    monkeypatch.delenv("TARDIS_PACKED_MAX")
    monkeypatch.delenv("TARDIS_PREFILL_MIN")
    monkeypatch.setenv("TARDIS_DECODE_THREADS", "512")     # (decode blocks of 512 threads read no one-byte codes)
    few = memory(16)
    monkeypatch.setenv("TARDIS_PACKED_MAX", "16")
    assert few == memory(16)


@pytest.mark.parametrize("max_batch,st", [(1, T.ERR_SHAPE), (5, T.ERR_SHAPE), (17, T.ERR_SHAPE), (18, T.OK)])
def test_single_launch_stacks_of_packed_layers(hip, monkeypatch, max_batch, st):  # noqa: F811
    """TARDIS_STACK_FUSED=2 refuses a stack that the single launch, which reads one-byte codes, is not for: packed layers are
    for it where they keep those for products, and one-token calls of the others read the packed codes."""
    monkeypatch.setenv("TARDIS_STACK_FUSED", "2")
    layers = [hip.fold(d=2048, h=2048, max_batch=max_batch, bits=4)[1] for _ in range(2)]
    call = hip.lib.tardis_stack_forward
    call.argtypes = [C.POINTER(C.c_void_p), C.c_int32, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p]
    got = call((C.c_void_p * 2)(*(L.value for L in layers)), 2, 1 << 38, 1, 1 << 37, None)
    for L in layers:
        hip.lib.tardis_destroy(L)
    assert got == st
