"""What tardis_fold and tardis_destroy do on the host, on a HIP runtime without a GPU (host_runtime.py): which memory they ask
for, keep and return, what they put into a stream that is being captured, and in which order."""
import pytest

from host_runtime import GIB, hip, host  # noqa: F401
from paper_2501_10054_amd import tardis as T


@pytest.mark.parametrize("opts", [{}, {"dtype": T.F32}, {"d": 1024, "h": 4096, "deterministic": 1}])
def test_a_fold_that_a_capture_refuses_leaves_nothing_in_it(hip, opts):
    """No memory can be asked for while a stream is captured, so the fold is refused; memory that the library keeps is no reason
    to record the fold's first steps, on memory that is returned or used again afterwards."""
    st, L = hip.fold(**opts)
    assert st == T.OK and hip.lib.tardis_destroy(L) == T.OK
    hip.events()
    hip.lib.fake_capture(1)
    st, L = hip.fold(**opts)
    assert st == T.ERR_HIP and not L.value
    assert not set(hip.events()) & {"set", "copy", "launch"}
    hip.lib.fake_capture(0)
    st, L = hip.fold(**opts)
    assert st == T.OK and hip.lib.tardis_destroy(L) == T.OK
    assert not set(hip.events()) & {"wild-free", "wild-write"}


def test_a_layer_destroyed_during_a_capture_does_not_spoil_it(hip):
    """To wait for the device ends every capture in progress; whoever destroys a layer meanwhile need not know of one."""
    layers = [hip.fold(d=512, h=2048 + 512 * k)[1] for k in range(6)]
    hip.lib.fake_capture(1)
    for L in layers:
        assert hip.lib.tardis_destroy(L) == T.OK
    hip.lib.fake_capture(0)
    assert not hip.lib.fake_broken()


def test_kept_memory_is_written_only_after_the_device_was_idle(hip):
    """A caller may have left work on a layer's memory under way."""
    L = hip.fold()[1]
    hip.lib.tardis_destroy(L)
    hip.events()
    st, L = hip.fold()
    events = hip.events()
    assert st == T.OK and "sync" in events and events.index("sync") < min(events.index(e) for e in ("set", "copy", "launch"))
    hip.lib.tardis_destroy(L)


def _bytes(hip, **opts):
    """device memory of a layer"""
    before = hip.lib.fake_used()
    st, L = hip.fold(**opts)
    assert st == T.OK
    return hip.lib.fake_used() - before, L


@pytest.mark.parametrize("sizes", [[300 << 20] * 8, [1 << 20] * 40, [900 << 20, 100 << 20, 3 << 20]])
def test_one_destroyed_layer_is_kept(hip, sizes):
    """Whatever is destroyed, the library holds the memory of the last one at most, and none of more than 1 GiB."""
    h = [max(64, size // (5 * 1024) // 64 * 64) + 64 * k for k, size in enumerate(sizes)]
    layers = [_bytes(hip, d=1024, h=v) for v in h]
    for size, L in layers:
        assert hip.lib.tardis_destroy(L) == T.OK
    assert hip.lib.fake_used() == layers[-1][0]
    big, L = _bytes(hip, d=8192, h=32768)
    kept = hip.lib.fake_used() - big
    assert big > GIB and hip.lib.tardis_destroy(L) == T.OK and hip.lib.fake_used() == kept
    assert "wild-free" not in hip.events()


def test_release_memory(hip):
    for k in range(3):
        hip.lib.tardis_destroy(hip.fold(h=2048 + 512 * k)[1])
    assert hip.lib.fake_used() > 0
    assert hip.lib.tardis_release_memory() == T.OK and hip.lib.fake_used() == 0
    assert hip.lib.tardis_release_memory() == T.OK


def test_nothing_is_kept_where_memory_is_short(hip):
    """A program that destroys a layer while less than half of the device is free gets its memory back."""
    for spare, kept in ((-4096, False), (4096, True)):
        size, L = _bytes(hip)
        hip.lib.fake_reset(2 * size + spare)
        hip.lib.tardis_destroy(L)
        assert hip.lib.fake_used() == (size if kept else 0)
        hip.lib.fake_reset(288 * GIB)


def test_an_allocation_that_fails_returns_what_is_kept(hip):
    size, L = _bytes(hip, h=2560)
    more, M = _bytes(hip, h=4096)
    hip.lib.tardis_destroy(L)
    hip.lib.tardis_destroy(M)
    assert hip.lib.fake_used() == more
    hip.lib.fake_reset(more + size // 2)              # room for a layer of the other size, but not beside what is kept
    st, L = hip.fold(h=2560)
    assert st == T.OK and hip.lib.fake_used() == size
    hip.lib.fake_reset(288 * GIB)
    hip.lib.tardis_destroy(L)
    hip.lib.fake_reset(more)                          # and no room for this one
    st, L = hip.fold(d=1024, h=8192, max_batch=4096)
    assert st == T.ERR_OOM and not L.value and hip.lib.fake_used() == 0


def test_kept_memory_stays_on_its_device(hip):
    size, L = _bytes(hip)
    hip.lib.tardis_destroy(L)
    hip.lib.fake_device(1)
    other, M = _bytes(hip)
    assert other == size                              # not the first device's block
    hip.lib.fake_device(0)
    again, L = _bytes(hip)
    assert again == 0                                 # that one
    hip.lib.tardis_destroy(M)                         # from the wrong device: freed
    assert hip.lib.fake_used() == size
    hip.lib.tardis_destroy(L)
