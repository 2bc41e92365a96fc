"""The one-sided rounding of the matrix cores must not survive the contractions.  They align the
terms of one instruction by rounding towards minus infinity, so that every sum comes out a
little low; stages contracted with alternating signs and, in the synthesis, rings of
alternating sign take the effect out of the means.  An iteration adds the error of a transform to
the iterate again and again, so what matters is not its size but the part that repeats: its
mean.

Statistic: mean / rms of the error of one transform against the FP64 path, over the real and
imaginary parts of the coefficients (analysis) or of the Fourier coefficients of the equatorial
rings (synthesis).  With the signs fixed it is -0.24 (nside 64) to -0.31 (nside 256) in the
analysis and -0.14 to -0.18 in the synthesis (measured on kernels with the alternation taken out); an
unbiased error of n = 5e4 values or more has |mean| / rms of n^-1/2 < 0.005, and what the alternation
leaves is 0.03 at most.  The bound is 0.08, little over half the smallest figure with fixed
signs."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_4931_amd import mfwf
    mfwf.load()
    return mfwf


def ratio(e):
    return float(e.mean() / e.pow(2).mean().sqrt())


def belt_coefficients(m, nside, lmax):
    """F(m') = sum_j m_j exp(-i m' phi_j) of the rings of 4 nside pixels, m' = 1 .. lmax"""
    n = 4 * nside
    start = 2 * nside * (nside - 1)
    rings = m[:, start:start + (2 * nside + 1) * n].reshape(m.shape[0], 2 * nside + 1, n)
    k = torch.arange(1, min(lmax, n // 2 - 1) + 1, device=m.device, dtype=torch.float64)
    i = torch.arange(2 * nside + 1, device=m.device)
    phi0 = torch.where(i % 2 == 0, np.pi / n, 0.0)  # half a pixel on every other ring, the first among them
    f = torch.fft.rfft(rings)[..., 1:k.numel() + 1]
    return f * torch.polar(torch.ones_like(f.real[0]), -phi0[:, None] * k[None])


# 32-column tiles as the small launches take them, the wide ones, and lambda generated
@pytest.mark.parametrize("nside,spec", [(64, ""), (64, "cta=2,cts=2,lamgen=1"), (256, "cta=1,cts=1,lamgen=0"), (256, "cta=2,cts=2,lamgen=0")])
def test_errors_of_the_contractions_have_no_sign(mf, nside, spec):
    lmax, maps = 2 * nside, 3
    g = torch.Generator(device="cuda").manual_seed(nside)
    d = torch.randn(maps, 12 * nside * nside, generator=g, dtype=torch.float64, device="cuda")
    p64 = mf.Plan(nside, lmax, max_batch=maps)
    if spec:
        os.environ["MFWF_TUNE_FORCE"] = spec
    try:
        p32 = mf.Plan(nside, lmax, max_batch=maps, dtype="f32")
    finally:
        os.environ.pop("MFWF_TUNE_FORCE", None)
    a = p64.sht_fwd(d)
    ana = ratio(torch.view_as_real(p32.sht_fwd(d) - a)[:, lmax + 1:])  # m > 0: both parts
    e = belt_coefficients(p32.sht_inv(a) - p64.sht_inv(a), nside, lmax)
    syn = ratio(torch.view_as_real(e))
    print("nside %d %s: analysis %.4f synthesis %.4f" % (nside, spec, ana, syn))
    assert abs(ana) < 0.08 and abs(syn) < 0.08
