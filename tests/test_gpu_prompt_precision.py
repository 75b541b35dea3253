"""Calls with many tokens keep the bits that calls with few have, also where what is added up cancels or is large."""
import numpy as np
import pytest
import torch

from paper_2501_10054_amd import synth
from paper_2501_10054_amd import tardis as T
from test_gpu_parity import DEV, dev, host, rel_l2

pytestmark = pytest.mark.gpu


def _layer(W1, W2, lo, hi, a, c, n, **kw):
    full = lambda v: torch.full((W1.shape[0],), v, dtype=torch.float32, device=DEV)
    return T.tardis_fold(T.FFN(dev(W1, "bf16"), dev(W2, "bf16")), full(lo), full(hi), full(a), full(c), max_batch=n, **kw)


@pytest.mark.parametrize("d,h,n", [(512, 2048, 65), (1024, 4096, 200), (768, 3080, 333), (2048, 8192, 700)])
def test_terms_of_the_folded_matrix_that_cancel(d, h, n):
    """Neurons in pairs with W1 rows r and r (1 + 2^-6 s) and opposite W2 columns: the sum over the neurons of a W1_j W2_j is about
    2^-6 of its terms.  W' is that sum, rounded once: y is off by its own rounding and that of W', 2^-9 each at most
    (r.m.s. 2^-9 / sqrt(3) and a little more), 1.6e-3 to 2.3e-3 together; the sum of the terms, each rounded to bf16, is off by 0.15."""
    rng = np.random.default_rng(23)
    half = h // 2
    as16 = lambda v: torch.from_numpy(np.asarray(v, np.float32)).bfloat16().float().numpy()
    r = as16(rng.standard_normal((half, d)) * d ** -0.5)
    W1 = np.concatenate([r, as16(r * (1.0 + 2.0 ** -6 * rng.choice([-1.0, 1.0], (half, 1))))])
    w2 = as16(rng.standard_normal((d, half)) * 0.05)
    W2 = np.concatenate([w2, -w2], axis=1)
    L = _layer(W1, W2, -1e9, 1e9, 0.7, 0.0, n)
    X = synth.make_tokens(n, d, "bf16", synth.workload_seed(9, 110), synth.STREAM_TEST)
    got = host(T.tardis_ffn_forward_batched(L, dev(X, "bf16")))
    L.close()
    a = float(np.float32(0.7))
    want = a * (X.astype(np.float64) @ W1.T.astype(np.float64)) @ W2.T.astype(np.float64)
    assert rel_l2(got, want) <= 3e-3


@pytest.mark.parametrize("n", [65, 300])
def test_pre_activations_beyond_32_bits_that_nothing_flagged(n):
    """Pre-activations of 1e40 with ranges that hold everything: y is W'x, whose weights and sums are ordinary numbers."""
    d, h = 512, 2048
    rng = np.random.default_rng(24)
    W1, W2 = (torch.from_numpy((rng.standard_normal(s) * k).astype(np.float32)).bfloat16().float().numpy() for s, k in (((h, d), 1e20), ((d, h), 1e-20)))
    L = _layer(W1, W2, -float("inf"), float("inf"), 0.5, 0.0, n)
    X = (synth.make_tokens(n, d, "bf16", synth.workload_seed(9, 111), synth.STREAM_TEST)).astype(np.float64)
    X = torch.from_numpy(X * 1e20).bfloat16().double().numpy()
    got = host(T.tardis_ffn_forward_batched(L, dev(X, "bf16")))
    mask, _, _ = T.tardis_get_last_outliers(L, n, want_list=False)
    L.close()
    assert not mask.any()
    want = 0.5 * (X @ W1.T.astype(np.float64)) @ W2.T.astype(np.float64)
    assert rel_l2(got, want) <= 1e-2


@pytest.mark.parametrize("d,h,bits", [(1024, 4096, 8), (2048, 2048, 8), (2048, 2048, 4), (4096, 2048, 8), (4096, 2048, 4)])
@pytest.mark.parametrize("n", [5, 16, 17])
def test_up_to_17_tokens_have_repair_factors_of_32_bits(d, h, bits, n):
    """Factors that have to cancel against b', as in test_repair_factors_are_not_rounded_to_one_bf16 (one bf16 a factor: 2 to 6 %), for
    layers whose calls of more tokens round them."""
    seed = synth.workload_seed(9, 112)
    layer = synth.make_layer(d, h, "bf16", seed, w1_std=d ** -0.5, w2_std=0.05, heavy_frac=0.0, with_bias=False)
    L = _layer(layer.W1, layer.W2, 0.0, 0.0, 0.0, 16.0, n, sketch_bits=bits)
    X = synth.make_tokens(n, d, "bf16", seed, synth.STREAM_TEST)
    got = host(T.tardis_ffn_forward_batched(L, dev(X, "bf16")))
    L.close()
    z = torch.from_numpy(X).double() @ torch.from_numpy(layer.W1).double().T
    want = (torch.nn.functional.gelu(z) @ torch.from_numpy(layer.W2).double().T).numpy()
    assert rel_l2(got, want) <= 3e-3
