"""The products with four wavefronts (large tiles): the folded and the dense path against the oracle at tokens on the
edges of their tiles, the fold and the calibration at partial tiles."""
import numpy as np
import pytest
import torch

from oracle import tardis_oracle as O
from paper_2501_10054_amd import synth
from paper_2501_10054_amd import tardis as T
from test_gpu_parity import DEV, assert_y_close, custom_layer, dev, host, make_ffn, rel_l2, unpack_mask

pytestmark = pytest.mark.gpu


# d, h, tokens: tiles of the predictor's and the hidden product, and of the two paths' output products (test_tile_choice holds the library
# to them)
TILES = {(2048, 2056, 769): ("128x128", "128x128 of eight", "128x128 ragged", "128x128 ragged"),
         (4096, 2056, 1537): ("192x128", "192x128", "256x256 ragged", "256x128 ragged"),
         (4096, 4104, 1500): ("256x128", "256x128", "192x256 ragged", "192x128 ragged"),
         (4096, 4104, 2048): ("192x256", "192x256", "256x256 ragged", "256x128 ragged"),
         (2048, 8192, 1537): ("256x256", "256x256", "256x128", "256x128"),
         (3072, 6152, 1500): ("192x256 of eight", "192x256 of eight", "192x256 ragged", "192x256 ragged"),
         (4096, 6152, 1537): ("192x128", "192x128", "256x256 ragged", "256x256 ragged")}


@pytest.mark.parametrize("d,h,n,act", [(*size, act) for size, act in zip(TILES, ("gelu_erf", "gelu_tanh", "relu", "gelu_erf", "gelu_erf", "gelu_erf", "gelu_tanh"))])
def test_tokens_on_the_edges_of_large_tiles(d, h, n, act):
    """Whole and ragged K (h = 2056, 4104), partial rows and columns of tiles; every mask word, y at the first and last
    rows of tiles and in the last, partial one.  The dense path against fp64 with its hidden activations rounded
    to bf16: as in test_prompt_path_tiles_of_128_columns."""
    seed = synth.workload_seed(9, 90)
    layer = custom_layer(d, h, "bf16", seed, 0.02, True)
    ffn = make_ffn(layer, act)
    X = synth.make_tokens(n, d, "bf16", seed, synth.STREAM_TEST)
    ranges = T.tardis_calibrate(ffn, dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), 0.93)
    L = T.tardis_fold(ffn, *ranges, max_batch=n)
    x = dev(X, "bf16")
    y = T.tardis_ffn_forward_batched(L, x)
    mask, _, _ = T.tardis_get_last_outliers(L, n, want_list=False)
    dense = T.tardis_dense_forward(L, x)
    at = sorted({0, 15, 127, 128, 191, 192, 255, 256, n // 2, (n - 1) // 64 * 64, n - 1})
    F = O.build(layer.W1, layer.b1, layer.W2, layer.b2, *(t.cpu().numpy() for t in ranges), act)
    want, flags = O.forward(F, X[at])
    got_flags = unpack_mask(mask, h)
    assert np.array_equal(got_flags[at], flags)
    assert 0 < got_flags.mean() < 0.2 and got_flags.any(0).mean() > 0.9 and got_flags.any(1).all()
    assert_y_close(host(y[at]), want, F, X[at], flags)
    W1, W2, b1, b2 = (torch.from_numpy(np.asarray(t)).double() for t in (layer.W1, layer.W2, layer.b1, layer.b2))
    z = torch.from_numpy(X[at]).double() @ W1.T + b1
    sigma = {"gelu_erf": torch.nn.functional.gelu, "gelu_tanh": lambda v: torch.nn.functional.gelu(v, approximate="tanh"),
             "relu": torch.relu}[act]
    ref = (sigma(z).to(torch.bfloat16).double() @ W2.T + b2).numpy()
    assert rel_l2(host(dense[at]), ref) <= 3e-3
    assert np.abs(host(dense[at]) - ref).max() <= 2.0 ** -7 * np.abs(ref).max()
    L.close()


@pytest.mark.parametrize("d,h,n", [(640, 8200, 1500), (1024, 4104, 1537)])
def test_fold_and_calibration_on_large_tiles(d, h, n):
    """Pre-activations (ragged rows, bias per row) and the fold's two products (ragged K, the second added to the first)."""
    seed = synth.workload_seed(9, 91)
    layer = custom_layer(d, h, "bf16", seed, 0.02, True)
    ffn = make_ffn(layer)
    X = synth.make_tokens(n, d, "bf16", seed, synth.STREAM_CAL)
    got = [host(t) for t in T.tardis_calibrate(ffn, dev(X, "bf16"), 0.9)]
    rows = np.r_[0:40, h // 2:h // 2 + 40, h - 40:h]
    want = O.calibrate(layer.W1[rows], layer.b1[rows], X, 0.9, "gelu_erf")
    scale = np.abs(np.concatenate(want[:2])).max()
    for g, w, tol in zip(got, want, (2e-5 * scale, 2e-5 * scale, 5 / n + 1e-4, 5 / n + 1e-4)):
        assert np.abs(g[rows] - w).max() <= tol
    L = T.tardis_fold(ffn, *(torch.from_numpy(g).float().to(DEV) for g in got), max_batch=1)
    Wp, _ = T.tardis_get_folded(L)
    ref = (np.asarray(layer.W2, np.float64) * got[2].astype(np.float32)) @ np.asarray(layer.W1, np.float64)
    assert rel_l2(host(Wp), ref) <= 3e-3
    # one rounding to bf16 (2^-9 of the value, or of the binade's bottom) of sums off by 2^-16 of their terms
    terms = np.sqrt((np.asarray(layer.W2, np.float64) ** 2 * got[2] ** 2) @ np.asarray(layer.W1, np.float64) ** 2)
    assert (np.abs(host(Wp) - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -14 * terms).all()
    L.close()


@pytest.mark.parametrize("d,h", [(130, 136), (257, 264), (132, 520), (640, 1032), (75, 130)])
def test_fold_rounds_in_the_second_product(d, h):
    """Rows that are and are not whole vectors of four (and, the last one, products on the kernel for any shape): W' within
    one rounding of the sums, and both copies of W2 (one token through the dense and through the folded layer)."""
    seed = synth.workload_seed(9, 92)
    layer = custom_layer(d, h, "bf16", seed, 0.1, True)
    ffn = make_ffn(layer)
    X = synth.make_tokens(3, d, "bf16", seed, synth.STREAM_TEST)
    ranges = T.tardis_calibrate(ffn, dev(synth.make_tokens(256, d, "bf16", seed, synth.STREAM_CAL), "bf16"), 0.9)
    L = T.tardis_fold(ffn, *ranges, max_batch=3)
    a = ranges[2].cpu().numpy().astype(np.float64)
    W1, W2 = (np.asarray(t, np.float64) for t in (layer.W1, layer.W2))
    ref, terms = (W2 * a) @ W1, np.sqrt((W2 ** 2 * a ** 2) @ W1 ** 2)
    got = host(T.tardis_get_folded(L)[0])
    assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -14 * terms).all()
    F = O.build(layer.W1, layer.b1, layer.W2, layer.b2, *(t.cpu().numpy() for t in ranges))
    want, flags = O.forward(F, X)
    assert_y_close(host(T.tardis_ffn_forward_batched(L, dev(X, "bf16"))), want, F, X, flags)
    z = torch.from_numpy(X).double() @ torch.from_numpy(W1).T + torch.from_numpy(np.asarray(layer.b1)).double()
    dense = (torch.nn.functional.gelu(z) @ torch.from_numpy(W2).T).numpy() + np.asarray(layer.b2, np.float64)
    assert rel_l2(host(T.tardis_dense_forward(L, dev(X, "bf16"))), dense) <= 1e-2
    L.close()
