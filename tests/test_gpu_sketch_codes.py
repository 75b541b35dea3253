"""Predictor codes taken in fp32 where that decides them: quotients at and beside halves, rows outside fp32's comfort, widths around
what a thread keeps; and the folded bias with rows of a last, incomplete block."""
import numpy as np
import pytest
import torch

from oracle import tardis_oracle as O
from paper_2501_10054_amd import tardis as T

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _weights(h, d, dtype, seed):
    """Rows of normal weights, of exact halves of their unit, of fp32 neighbours of halves, tiny, huge, nearly zero and zero ones."""
    gen = torch.Generator().manual_seed(seed)
    W = torch.randn(h, d, generator=gen) * 0.02
    half = (torch.randint(-127, 127, (h, d), generator=gen) + 0.5).clamp(-127, 127)
    W[1::8] = half[1::8] / 64
    W[2::8] = torch.nextafter(half[2::8], torch.randn(h, d, generator=gen)[2::8] * 1e9)
    W[3::8] = half[3::8] * 1.3e-3
    for r in (1, 2, 3):                                              # (the row's largest: one unit is 1/64, 1, 1.3e-3)
        W[r::8, 0] = 127.0 * (1 / 64, 1.0, 1.3e-3)[r - 1]
    W[4::8] *= 1e-33
    W[5::8] *= 1e34
    W[6::8, 1:] *= 1e-4
    W[7::16] = 0.0
    W[:, 32:64] *= (torch.arange(h) % 3 != 0)[:, None]               # empty groups
    return W.to(dtype)


def _codes(W, bits):
    h, d = W.shape
    ffn = T.FFN(W.to(DEV), torch.zeros(d, h, dtype=W.dtype, device=DEV))
    full = lambda v: torch.full((h,), v, device=DEV)
    L = T.tardis_fold(ffn, full(-0.1), full(0.2), full(0.0), full(0.0), sketch_bits=bits)
    Q, tlo, thi = (t.cpu().numpy() for t in T.tardis_get_predictor_state(L))
    m = None if bits == 8 else T.tardis_get_sketch_groups(L).cpu().numpy()
    L.close()
    return Q, tlo, thi, m


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("bits", [8, 4, 3, 2])
@pytest.mark.parametrize("d", [32, 96, 4096, 4128])
def test_codes_are_the_exact_quotients(d, bits, dtype):
    h = 62
    W = _weights(h, d, dtype, d + bits)
    Q, tlo, thi, m = _codes(W, bits)
    lo, hi = np.full(h, -0.1, np.float32), np.full(h, 0.2, np.float32)
    want = O.sketch(W.double().numpy(), None, lo, hi, bits=bits)
    np.testing.assert_array_equal(Q, want.Q)
    np.testing.assert_array_equal(tlo, want.tlo)
    np.testing.assert_array_equal(thi, want.thi)
    if bits != 8:
        np.testing.assert_array_equal(m, want.m)


@pytest.mark.parametrize("bits", [8, 4])
def test_codes_of_rows_that_are_not_finite(bits):
    """A zero column more is a width that takes every quotient in 64 bits: NaNs and infinities get the same codes there."""
    h, d = 32, 96
    W = _weights(h, d, torch.float32, 5)
    W[0::4, 7] = float("nan")
    W[1::4, 40] = float("inf")
    W[2::8, 90] = -float("inf")
    W[3, :] = float("nan")
    Q, tlo, thi, m = _codes(W, bits)
    Q1, tlo1, thi1, m1 = _codes(torch.cat([W, torch.zeros(h, 1)], 1), bits)
    np.testing.assert_array_equal(Q, Q1[:, :d])
    np.testing.assert_array_equal(tlo, tlo1)
    np.testing.assert_array_equal(thi, thi1)
    if bits != 8:
        np.testing.assert_array_equal(m, m1[:, :d // 32])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,h", [(33, 40), (34, 4104), (39, 65), (64, 2048)])
def test_folded_bias(d, h, dtype):
    gen = torch.Generator(device=DEV).manual_seed(d)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=gen)
    W1, W2, b1, b2 = (t.to(dtype) for t in (rnd(h, d) * 0.1, rnd(d, h) * 0.1, rnd(h), rnd(d)))
    a, c = rnd(h), rnd(h)
    L = T.tardis_fold(T.FFN(W1, W2, b1, b2), -torch.ones_like(a), torch.ones_like(a), a, c)
    got = T.tardis_get_folded(L)[1].double()
    L.close()
    k = c.double() + a.double() * b1.double()
    want = W2.double() @ k + b2.double()
    # 64-bit sums rounded once to fp32
    assert ((got - want).abs() <= 2.0 ** -24 * want.abs() + 1e-13 * (W2.double().abs() @ k.abs())).all()
