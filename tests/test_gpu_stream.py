"""Calls of up to 64 tokens whose products stream the weights: masks bit for bit and y against the oracle at the edges of the tiles (32 and
64 rows of the weights, 32 and 64 tokens), and rows of W1 that have no scale for their codes or only zeros."""
import numpy as np
import pytest
import torch

from oracle import tardis_oracle as O
from paper_2501_10054_amd import synth
from paper_2501_10054_amd import tardis as T
from test_gpu_parity import DEV, assert_y_close, custom_layer, dev, host, make_ffn, rel_l2, unpack_mask

pytestmark = pytest.mark.gpu


# d, h, tokens: matrix products of a call (test_stream_choice holds the library to them).  "repair 32 x 64": up to 32 tokens, 64 rows of the
# weights a block; "repair", "part" alone: gemm_tile_kernel.  Layers without whole 2048s of neurons have a second output product, of the
# remainders of the factors; the dense path's output product is the last entry
STREAMS = {(1024, 1000, 19): ("repair 32 x 32", "part", "part", "part"),
           (1024, 8200, 32): ("repair 32 x 64", "part", "part", "part"),
           (2048, 1000, 64): ("repair 64 x 32", "part", "part", "part"),
           (2048, 8200, 33): ("repair 64 x 64", "part", "part", "part"),
           (4096, 3336, 32): ("repair 32 x 32", "part", "part", "part"),
           (4096, 3328, 19): ("repair 32 x 32", "part 32 x 64", "part", "part"),
           (4096, 3328, 64): ("repair 64 x 32", "part", "part", "part"),
           (4096, 8320, 40): ("repair 64 x 64", "part 64 x 64", "part", "part"),
           (4096, 10240, 34): ("repair 64 x 64", "part 64 x 64", "part"),
           (1024, 30720, 20): ("repair", "part 32 x 32", "part 32 x 32"),
           (2048, 14720, 32): ("repair 32 x 64", "part 32 x 64", "part 32 x 64", "part 32 x 64"),
           (4096, 3328, 33): ("repair 64 x 32", "part", "part", "part"),
           (128, 1000, 19): ("repair", "part", "part", "part"),
           (256, 8192, 32): ("repair", "part", "part", "part"),
           (128, 8200, 64): ("repair", "part", "part", "part"),
           (384, 16392, 33): ("repair", "part", "part", "part")}


def _check(layer, act, n, seed, d, h, coverage=0.85, bits=8, few=18, dense=False):
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
    if dense:                                         # (fp64 with the hidden activations rounded to bf16, as in test_prompt_path_tiles_of_128_columns)
        W1, W2, b1, b2 = (torch.from_numpy(np.asarray(t)).double() for t in (layer.W1, layer.W2, layer.b1, layer.b2))
        sigma = {"gelu_erf": torch.nn.functional.gelu, "gelu_tanh": lambda v: torch.nn.functional.gelu(v, approximate="tanh"), "relu": torch.relu}[act]
        ref = (sigma(torch.from_numpy(X).double() @ W1.T + b1).to(torch.bfloat16).double() @ W2.T + b2).numpy()
        got = host(T.tardis_dense_forward(L, dev(X, "bf16")))
        assert rel_l2(got, ref) <= 3e-3 and np.abs(got - ref).max() <= 2.0 ** -7 * np.abs(ref).max()
    L.close()


@pytest.mark.parametrize("d,h,n,act", [(*size, act) for size, act in zip(STREAMS, ("gelu_erf", "relu", "gelu_tanh", "gelu_erf", "gelu_erf", "gelu_erf", "gelu_erf",
                                                                                     "gelu_tanh", "relu", "gelu_erf", "gelu_tanh", "gelu_tanh", "gelu_erf", "gelu_tanh", "relu", "gelu_erf"))])
def test_streams_of_few_tokens(d, h, n, act):
    """Partial tiles of 32 and 64 rows, ranges of K, one and two output products, each as a stream and not."""
    seed = synth.workload_seed(9, 101)
    _check(custom_layer(d, h, "bf16", seed, 0.02 if d > 1000 else 0.1, True), act, n, seed, d, h, dense=True)


def test_streams_take_tokens_at_any_address():
    """Tokens and outputs that are not 16-byte aligned give the same bits, and so do the last tokens of a call in chunks."""
    d, h = 2048, 2048
    seed = synth.workload_seed(9, 105)
    layer = custom_layer(d, h, "bf16", seed, 0.02, True)
    ffn = make_ffn(layer)
    L = T.tardis_fold(ffn, *T.tardis_calibrate(ffn, dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), 0.85), max_batch=64)
    x = dev(synth.make_tokens(64, d, "bf16", seed, synth.STREAM_TEST), "bf16")
    for n in (18, 24, 32, 64):
        want = T.tardis_ffn_forward_batched(L, x[:n])
        mask = T.tardis_get_last_outliers(L, n, want_list=False)[0]
        buf = torch.zeros(n * d + 1, dtype=torch.bfloat16, device=DEV)
        out = torch.zeros_like(buf)
        buf[1:] = x[:n].flatten()
        got = T.tardis_ffn_forward_batched(L, buf[1:].view(n, d), out[1:].view(n, d))
        assert torch.equal(got, want) and torch.equal(T.tardis_get_last_outliers(L, n, want_list=False)[0], mask)
    L.close()


def test_chunks_of_a_long_call_that_stream(monkeypatch):
    """84 tokens in chunks of 64 and 20: the first one's up product is not a stream at d = 1024, the second one's is."""
    monkeypatch.setenv("TARDIS_PREFILL_CHUNK", "64")
    d, h, n = 1024, 2048, 84
    seed = synth.workload_seed(9, 106)
    _check(custom_layer(d, h, "bf16", seed, 0.02, True), "gelu_erf", n, seed, d, h)


def test_graph_capture_of_streams():
    """Both products as streams, captured once and replayed with eager work on other tokens in between."""
    d, h, n = 4096, 3328, 32
    seed = synth.workload_seed(9, 107)
    layer = custom_layer(d, h, "bf16", seed, 0.02, True)
    ffn = make_ffn(layer)
    L = T.tardis_fold(ffn, *T.tardis_calibrate(ffn, dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), 0.85), max_batch=n)
    x = dev(synth.make_tokens(n, d, "bf16", seed, synth.STREAM_TEST), "bf16")
    want = T.tardis_ffn_forward_batched(L, x).clone()
    masks = T.tardis_get_last_outliers(L, n, want_list=False)[0].clone()
    torch.cuda.synchronize()
    y = torch.zeros_like(want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        T.tardis_ffn_forward_batched(L, x, y)
    for _ in range(3):
        y.zero_()
        T.tardis_ffn_forward_batched(L, torch.roll(x, 1, 0).contiguous())
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(T.tardis_get_last_outliers(L, n, want_list=False)[0], masks)
    L.close()


@pytest.mark.parametrize("d,h,std", [(256, 1024, 0.1), (2048, 1024, 0.02)])
@pytest.mark.parametrize("tiny", [0.0, 2.0 ** -110])
def test_rows_without_a_scale(d, h, std, tiny):
    """Rows of zeros have codes of zero; a row below 1e-30 has no scale, and the layer's calls read its stored codes (as those of d = 256
    do anyway)."""
    n = 40
    seed = synth.workload_seed(9, 102)
    layer = custom_layer(d, h, "bf16", seed, std, True)
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
    d, h, n = 2048, 2048, 40
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
