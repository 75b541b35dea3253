"""Calls of up to 64 tokens whose products stream the weights: masks bit for bit and y against the oracle at the edges of the tiles (32 and
64 rows of the weights, 32 and 64 tokens), and rows of W1 that have no scale for their codes or only zeros."""
import numpy as np
import pytest
import torch

from oracle import tardis_oracle as O
from paper_2501_10054_amd import synth
from paper_2501_10054_amd import tardis as T
from test_gpu_parity import DEV, assert_y_close, custom_layer, dev, host, make_ffn, unpack_mask

pytestmark = pytest.mark.gpu


def _check(layer, act, n, seed, d, h, coverage=0.85, bits=8, few=18):
    ffn = make_ffn(layer, act)
    ranges = T.tardis_calibrate(ffn, dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), coverage)
    L = T.tardis_fold(ffn, *ranges, max_batch=n, sketch_bits=bits)
    X = synth.make_tokens(n, d, "bf16", seed, synth.STREAM_TEST)
    F = O.build(layer.W1, layer.b1, layer.W2, layer.b2, *(t.cpu().numpy() for t in ranges), act, **({} if bits == 8 else {"sketch_bits": bits}))
    for rows in sorted({n, max(few, n - 1)}):         # (and a call that leaves rows of the scratch from the one before)
        y = T.tardis_ffn_forward_batched(L, dev(X[:rows], "bf16"))
        mask, _, _ = T.tardis_get_last_outliers(L, rows, want_list=False)
        want, flags = O.forward(F, X[:rows])
        assert np.array_equal(unpack_mask(mask, h), flags)
        assert 0.05 < flags.mean() < 0.35
        assert_y_close(host(y), want, F, X[:rows], flags)
    L.close()


@pytest.mark.parametrize("d,h,n,act", [(128, 1000, 19, "gelu_erf"), (128, 8200, 64, "relu"), (256, 8192, 32, "gelu_tanh"), (384, 16392, 33, "gelu_erf"),
                                       (4096, 3328, 18, "gelu_erf"), (4096, 3328, 33, "gelu_tanh"), (4096, 3328, 64, "gelu_erf"),
                                       (4096, 3336, 32, "gelu_erf")])
def test_streams_of_few_tokens(d, h, n, act):
    """One slice of K and many, partial tiles of 32 and 64 rows, ranges of K; the output product as a stream (h = 3328) and not."""
    seed = synth.workload_seed(9, 101)
    _check(custom_layer(d, h, "bf16", seed, 0.02 if d > 1000 else 0.1, True), act, n, seed, d, h)


@pytest.mark.parametrize("tiny", [0.0, 2.0 ** -110])
def test_rows_without_a_scale(tiny):
    """Rows of zeros have codes of zero; a row below 1e-30 has no scale, and the layer's calls read its stored codes."""
    d, h, n = 256, 1024, 40
    seed = synth.workload_seed(9, 102)
    layer = custom_layer(d, h, "bf16", seed, 0.1, True)
    layer.W1[7] *= tiny
    layer.W1[1000] *= tiny
    _check(layer, "gelu_erf", n, seed, d, h)


@pytest.mark.parametrize("d", [2048, 4096])
@pytest.mark.parametrize("n", [4, 5, 8, 16, 17])
def test_packed_sketch_at_the_sizes_where_its_path_changes(d, n):
    """4-bit layers folded for up to 4 tokens keep the packed codes alone, for more one-byte codes as well (groups of 8 and 16; 4 tokens of a
    layer folded for 5 read either); 17 tokens are a group of 16 and one."""
    seed = synth.workload_seed(9, 103)
    _check(custom_layer(d, 2048, "bf16", seed, 0.02, True), "gelu_erf", n, seed, d, 2048, bits=4, few=1)


def test_rows_with_a_nan_have_the_stored_codes_on_every_path():
    """The predictor's code of a NaN is the definition's -127 in the stored codes; masks do not depend on how many tokens a call has."""
    d, h, n = 1024, 2048, 40
    seed = synth.workload_seed(9, 104)
    layer = custom_layer(d, h, "bf16", seed, 0.1, True)
    ranges = T.tardis_calibrate(make_ffn(layer), dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), 0.7)
    rng = np.random.default_rng(31)
    rows = rng.choice(h, 64, replace=False)
    for j in rows:
        layer.W1[j, rng.choice(d, 8, replace=False)] = np.nan
    L = T.tardis_fold(make_ffn(layer), *ranges, max_batch=n)
    x = dev(synth.make_tokens(n, d, "bf16", seed, synth.STREAM_TEST), "bf16")
    T.tardis_ffn_forward_batched(L, x)
    together = T.tardis_get_last_outliers(L, n, want_list=False)[0]
    one = []
    for t in range(n):
        T.tardis_ffn_forward(L, x[t].contiguous())
        one.append(T.tardis_get_last_outliers(L, 1, want_list=False)[0])
    assert torch.equal(together, torch.cat(one))
    L.close()
