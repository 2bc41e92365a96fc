"""Rings of all transform lengths in one launch (up to 2048 points, nside 256) and in two
(nside 512): the synthesis against the sum of spherical harmonics at the pixels of the shortest,
the longest chirp-z, the first and the last power-of-two rings, and of rings between, and the
analysis of the same rings as its adjoint.

Tolerance: sums of (lmax + 1)^2 = 441 terms of order one, FP64 transforms of log2(2048) = 11
stages twice (chirp-z), Legendre recurrences of 20 steps: a few hundred roundings, 1e-12 of
the largest value."""
import numpy as np
import pytest
import torch
from scipy.special import lpmv, gammaln

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_4931_amd import mfwf
    mfwf.load()
    return mfwf


def ring(nside, i):
    """(first pixel, cos theta, phi of its pixels) of ring i = 1 .. 4 nside - 1"""
    n = 4 * min(i, 4 * nside - i, nside)
    k = min(i, 4 * nside - i)
    if k < nside:
        z = 1.0 - k * k / (3.0 * nside * nside)
        z, shift = (z if i < 2 * nside else -z), 0.5
        start = 2 * k * (k - 1) if i < 2 * nside else 12 * nside * nside - 2 * k * (k + 1)
    else:
        z, shift = 4.0 / 3.0 - 2.0 * i / (3.0 * nside), 0.5 * ((i - nside + 1) % 2)
        start = 2 * nside * (nside - 1) + (i - nside) * 4 * nside
    return start, z, 2.0 * np.pi * (np.arange(n) + shift) / n


@pytest.mark.parametrize("nside,maps", [(2, 1), (64, 2), (128, 1), (256, 1), (256, 3), (512, 1)])
def test_rings_against_spherical_harmonics(mf, nside, maps):
    lmax = min(20, 2 * nside)
    rng = np.random.default_rng(nside)
    ms = np.concatenate([np.full(lmax + 1 - m, m) for m in range(lmax + 1)])
    ls = np.concatenate([np.arange(m, lmax + 1) for m in range(lmax + 1)])
    a = rng.standard_normal((maps, ms.size)) + 1j * rng.standard_normal((maps, ms.size))
    a[:, ms == 0] = a[:, ms == 0].real
    p = mf.Plan(nside, lmax, max_batch=maps)
    s = p.sht_inv(torch.as_tensor(a, device="cuda")).cpu().numpy()
    norm = np.sqrt((2 * ls + 1) / (4 * np.pi) * np.exp(gammaln(ls - ms + 1) - gammaln(ls + ms + 1)))
    w = np.where(ms == 0, 1.0, 2.0)
    t = np.zeros((maps, 12 * nside * nside))
    want = np.zeros((maps, ms.size), dtype=complex)
    for i in sorted({1, max(1, nside // 2), max(1, nside - 1), nside, nside + 1, 2 * nside,
                     4 * nside - 1, 3 * nside + nside // 2}):
        start, z, phi = ring(nside, i)
        y = (norm * lpmv(ms, ls, z))[:, None] * np.exp(1j * ms[:, None] * phi[None, :])
        ref = ((a * w) @ y).real
        assert np.abs(s[:, start:start + phi.size] - ref).max() <= 1e-12 * np.abs(ref).max()
        x = rng.standard_normal((maps, phi.size))
        t[:, start:start + phi.size] = x
        want += x @ y.conj().T
    got = p.sht_fwd(torch.as_tensor(t, device="cuda")).cpu().numpy() / (4 * np.pi / t.shape[1])
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
