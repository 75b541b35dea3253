"""The calibration's one-pass fit: lines through samples far from zero and close together, equal samples, few samples,
every activation, one to thirty-two samples a thread."""
import numpy as np
import pytest
import torch

from oracle import tardis_oracle as O
from paper_2501_10054_amd import tardis as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["gelu_erf", "gelu_tanh", "relu", "identity"])
@pytest.mark.parametrize("n", [2, 3, 64, 1025, 4096, 9000])
def test_lines_far_from_zero_and_equal_samples(act, n):
    """Rows 0-7: equal samples (zero weights, biases -8 to 40): slope 0, the intercept sigma of the bias.  Rows 8-39 (from 64
    samples on; fewer are the last test's): means of -6 to 6 and deviations down to a hundredth of them.  The pre-activations are fp32 sums of 16 products and a bias: off
    by at most 2^-21 of |z| + 1; a line through samples of deviation s moves by no more than 4 times that over s."""
    rng = np.random.default_rng(n)
    h, d = 40, 16
    W1 = rng.normal(0, 1, (h, d)).astype(np.float32) * np.r_[np.zeros(8), np.geomspace(0.01, 0.5, 32)][:, None].astype(np.float32)
    b1 = np.r_[np.linspace(-8, 40, 8), np.tile(np.linspace(-6, 6, 8), 4)].astype(np.float32)
    X = rng.normal(0, 1, (n, d)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ffn = T.FFN(dev(W1), torch.zeros(d, h, device="cuda"), dev(b1), None, act)
    lo, hi, a, c = (t.cpu().numpy().astype(np.float64) for t in T.tardis_calibrate(ffn, dev(X), 0.9))
    olo, ohi, oa, oc = O.calibrate(W1, b1, X, 0.9, act)
    z = X.astype(np.float64) @ W1.astype(np.float64).T + b1
    off = 2.0 ** -21 * (np.abs(z).max(0) + 1)
    assert (np.abs(lo - olo) <= off).all() and (np.abs(hi - ohi) <= off).all()
    assert (a[:8] == 0).all() and np.abs(c[:8] - O.act(b1[:8].astype(np.float64), act)).max() <= 2.0 ** -23 * 40
    inside = (z >= olo) & (z < ohi)
    compared = 0
    for j in range(8, h):
        zi = z[inside[:, j], j]
        near = (np.abs(z[:, j] - olo[j]) <= off[j]) | (np.abs(z[:, j] - ohi[j]) <= off[j])
        if len(zi) < 3 or near.any():               # (a sample may fall on either side of an end)
            continue
        compared += 1
        tol = 4 * off[j] / zi.std() + 2.0 ** -22
        assert abs(a[j] - oa[j]) <= tol, (j, a[j], oa[j], tol)
        assert abs(c[j] - oc[j]) <= tol * (np.abs(zi).max() + 1), (j, c[j], oc[j])
    assert n < 64 or compared >= 20, compared


@pytest.mark.parametrize("n", [300, 2000, 6000, 12000])
def test_a_far_sample_that_the_end_leaves_out(n):
    """Coverage 1: the smallest sample is the end itself, and where that is rounded up the sample lies outside.  It is 1000
    away here, the others vary by 0.001: sums around it would lose eight digits of their deviations.  Pre-activations are
    single products by one, exact, but for the far one's (-1000 - 1e-6, as fp32 -1000); the line is fp64's, rounded."""
    rng = np.random.default_rng(n)
    h, d = 8, 16
    W1 = np.zeros((h, d), np.float32)
    W1[:, :8], W1[:, 8] = np.eye(8), 1.0
    X = np.zeros((n, d), np.float32)
    X[:, :8] = 0.5 + 1e-3 * rng.normal(0, 1, (n, 8))
    X[n // 3, :8], X[n // 3, 8] = -1000.0, -1e-6
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ffn = T.FFN(dev(W1), torch.zeros(d, h, device="cuda"), None, None, "gelu_erf")
    lo, hi, a, c = (t.cpu().numpy().astype(np.float64) for t in T.tardis_calibrate(ffn, dev(X), 1.0))
    z = X.astype(np.float64) @ W1.astype(np.float64).T
    assert (lo == -1000.0).all() and (z.min(0) < lo).all() and (hi == z.max(0)).all()
    for j in range(h):
        zi = z[(z[:, j] >= lo[j]) & (z[:, j] < hi[j]), j]
        assert len(zi) == n - 2
        g, dz = O.act(zi, "gelu_erf"), zi - zi.mean()
        slope = (dz * g).sum() / (dz * dz).sum()
        # fp64 sums of deviations around a sample among them: 2^-53 of sigma over the deviation, far below one rounding to fp32
        assert abs(a[j] - slope) <= 2.0 ** -24 * abs(slope) + 1e-11, (j, a[j] - slope)
        assert abs(c[j] - (g.mean() - slope * zi.mean())) <= 2.0 ** -24 + 1e-11


@pytest.mark.parametrize("act", ["gelu_erf", "gelu_tanh", "relu", "identity"])
@pytest.mark.parametrize("n", [300, 12000])
def test_equal_samples_on_both_sides_of_an_end(n, act):
    """The two smallest samples are one number in fp32 and differ in fp64; the end, between them, leaves the lower one out.  The same
    at the upper end.  Pre-activations of the others are single products by one, exact."""
    rng = np.random.default_rng(n)
    h, d = 8, 16
    W1 = np.zeros((h, d), np.float32)
    W1[:, :8], W1[:, 8] = np.eye(8), 1.0
    X = np.zeros((n, d), np.float32)
    X[:, :8] = np.clip(rng.normal(0, 0.5, (n, 8)), -1.9, 1.9)
    for at, value in ((7, -2.0), (n - 9, 2.0)):
        X[at, :8], X[at, 8], X[at + 1, :8], X[at + 1, 8] = value, -3e-8, value, 3e-8
    coverage = 1.0 - 0.2 / (n - 1)                   # ends a tenth of the way between the two samples
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ffn = T.FFN(dev(W1), torch.zeros(d, h, device="cuda"), None, None, act)
    lo, hi, a, c = (t.cpu().numpy().astype(np.float64) for t in T.tardis_calibrate(ffn, dev(X), coverage))
    z = X.astype(np.float64) @ W1.astype(np.float64).T
    assert (lo == -2.0).all() and (hi == 2.0).all()
    for j in range(h):
        zi = z[(z[:, j] >= lo[j]) & (z[:, j] < hi[j]), j]
        assert len(zi) == n - 2
        g, dz = O.act(zi, act), zi - zi.mean()
        slope = (dz * g).sum() / (dz * dz).sum()
        # one rounding to fp32, and the two samples at the ends as fp32 has them: 3e-8 in n numbers of deviation 0.5
        assert abs(a[j] - slope) <= 2.0 ** -24 * abs(slope) + 1e-8, (j, a[j] - slope)
        assert abs(c[j] - (g.mean() - slope * zi.mean())) <= 2.0 ** -24 + 1e-8


@pytest.mark.parametrize("act", ["gelu_erf", "gelu_tanh", "relu", "identity"])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_no_one_and_two_samples_inside(n, act):
    """Coverage 0.9 of n samples leaves n - 2 inside: no line but a constant, sigma(lo) without any and sigma(z) of one; two make the
    line through them.  Pre-activations are single products by one, exact."""
    rng = np.random.default_rng(10 + n)
    h = d = 40
    X = rng.normal(0, 1.5, (n, d)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ffn = T.FFN(dev(np.eye(h, dtype=np.float32)), torch.zeros(d, h, device="cuda"), None, None, act)
    lo, hi, a, c = (t.cpu().numpy().astype(np.float64) for t in T.tardis_calibrate(ffn, dev(X), 0.9))
    for j in range(h):
        z = X[:, j].astype(np.float64)
        zi = z[(z >= lo[j]) & (z < hi[j])]
        assert len(zi) == max(n - 2, 0)
        if len(zi) < 2:
            want = 0.0, O.act(zi if len(zi) else np.array([lo[j]]), act)[0]
        else:
            g = O.act(zi, act)
            slope = (g[1] - g[0]) / (zi[1] - zi[0])
            want = slope, g.mean() - slope * zi.mean()
        for got, w in zip((a[j], c[j]), want):
            assert abs(got - w) <= 2.0 ** -24 * abs(w) + 1e-13 * (1 + 1 / (np.ptp(zi) if len(zi) == 2 else 1)), (j, got, w)
