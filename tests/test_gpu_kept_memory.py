"""Memory of destroyed layers that the library keeps for the next fold: whatever it held does not show, it is bounded,
threads with their own streams share it."""
import threading

import pytest
import torch

from paper_2501_10054_amd import tardis as T

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _layer(d, h, seed, max_batch, **opts):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=gen)
    ffn = T.FFN((rnd(h, d) * 0.03).bfloat16(), (rnd(d, h) * 0.03).bfloat16())
    w = 1.9 * 0.03 * d ** 0.5
    full = lambda v: torch.full((h,), v, device=DEV)
    return T.tardis_fold(ffn, full(-w), full(w), full(0.5), full(0.1), max_batch=max_batch, **opts), rnd(max_batch, d).bfloat16()


def _results(d, h, seed, max_batch, **opts):
    L, x = _layer(d, h, seed, max_batch, **opts)
    out = []
    for n in (1, 3, 16, max_batch):
        y = T.tardis_ffn_forward_batched(L, x[:n].contiguous())
        mask, counts, _ = T.tardis_get_last_outliers(L, n, want_list=False)
        out.append((y.float(), mask.clone(), counts.clone()))
    out.append((T.tardis_dense_forward(L, x).float(),))
    torch.cuda.synchronize()
    L.close()
    return out


def _same(got, want):
    for g, w in zip(got, want):
        # groups of tokens add in fp32 atomics: a sum may round to the neighbouring bf16 number (2^-7 of it, or of the row's scale)
        assert ((g[0] - w[0]).abs() <= 2.0 ** -7 * w[0].abs() + 2.0 ** -12 * w[0].abs().max()).all()
        assert all(torch.equal(a, b) for a, b in zip(g[1:], w[1:]))


@pytest.mark.parametrize("opts", [{}, {"sketch_bits": 4}, {"deterministic": True}, {"folded_fp8": True}])
@pytest.mark.parametrize("d,h", [(1024, 4096), (768, 2000)])
def test_what_a_destroyed_layer_left_does_not_show(d, h, opts):
    if "deterministic" in opts and d == 768:
        pytest.skip("the ordered path exists for layers with decode kernels")
    want = _results(d, h, 1, 40, **opts)
    for seed in (2, 3):
        _results(d, h, seed, 40)                     # the same size, other contents and options
        _same(_results(d, h, 1, 40, **opts), want)


@pytest.mark.parametrize("d,h,count", [(4096, 12288, 8), (512, 2048, 24)])
def test_what_is_kept_is_one_layer_and_comes_back(d, h, count):
    """Eight layers of 290 to 460 MB, 24 of 6 to 70 MB, no two of a size: all destroyed, one stays with the library, and that
    until tardis_release_memory."""
    T.tardis_release_memory()
    layers = [_layer(d, h + 1024 * k, k, 2)[0] for k in range(count)]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    full, total = torch.cuda.mem_get_info()
    for L in layers:
        L.ffn = None                                  # (its weights are torch's)
        L.close()
    torch.cuda.empty_cache()
    left, _ = torch.cuda.mem_get_info()
    T.tardis_release_memory()
    free, _ = torch.cuda.mem_get_info()
    size = lambda k: 5 * d * (h + 1024 * k) + 2 * d * d       # two copies of W2 in bf16, codes, the folded matrix
    assert free - full >= sum(size(k) for k in range(count))
    assert free - left <= size(count - 1) + (64 << 20), (free, left)
    assert free - left >= size(count - 1) or left < total // 2
    again, x = _layer(d, h, 1, 2)
    T.tardis_ffn_forward_batched(again, x)
    again.close()
    T.tardis_release_memory()


def test_threads_with_streams_of_their_own():
    want = {seed: _results(1024, 4096, seed, 20) for seed in (5, 6)}
    errors = []

    def work(seed):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    _same(_results(1024, 4096, seed, 20), want[seed])
        except Exception as e:                       # noqa: BLE001 - reported by the test
            errors.append(e)

    threads = [threading.Thread(target=work, args=(seed,)) for seed in want]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_a_layer_destroyed_during_a_capture():
    """By the C call: Layer.close() waits for the device, which no capture survives."""
    keep, x = _layer(1024, 4096, 7, 2)
    gone, _ = _layer(1024, 4096, 8, 2)
    want = T.tardis_ffn_forward_batched(keep, x).clone()
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=stream):
        y = T.tardis_ffn_forward_batched(keep, x)
        assert T.lib().tardis_destroy(gone.handle) == T.OK
        gone.handle = None
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        # one token's or two tokens' sums, rounded to bf16 (see _same)
        assert ((y.float() - want.float()).abs() <= 2.0 ** -7 * want.float().abs() + 2.0 ** -12 * want.float().abs().max()).all()
        again, x2 = _layer(1024, 4096, 9, 2)         # (on the memory of the destroyed one)
        T.tardis_ffn_forward_batched(again, x2)
        torch.cuda.synchronize()
        again.close()
    keep.close()
